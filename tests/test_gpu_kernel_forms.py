"""Two forms of one kernel that a rule chooses between have to agree where the
rule may choose either, and keep what the general form accepts."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from paper_1806_09907_amd import api, synth, tune
from paper_1806_09907_amd._lib import lib
from parity import VAL_TOL, check_grad
from test_gpu_walk_edges import test_conv_linear_blocks as check_conv
from test_gpu_walk_edges import test_field_contractions as check_contraction

pytestmark = pytest.mark.gpu
DEV = "cuda"


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


# The squarings of a field that moves less than one voxel read their samples
# from LDS, the others from memory. One voxel of the second field moves two
# voxels, which sends its second squaring to memory; it reaches no sample more
# than a few voxels away, and there both squarings have the same inputs: the
# results must have the same bits.
@pytest.mark.parametrize("n", [(41, 27, 33), (34, 40, 21), (300, 37), (45, 70)])
def test_squaring_from_lds_and_from_memory_bitwise(n):
    d = len(n)
    rng = np.random.default_rng(11)
    th = rng.uniform(-1.6, 1.6, (d,) + tuple(reversed(n)))   # u_0 = theta / 4 in voxels
    far = th.copy()
    far[(0,) + (0,) * d] = 8.0
    for a in range(d):
        th[a] *= 2.0 / (n[a] - 1)
        far[a] *= 2.0 / (n[a] - 1)
    plan = api.Plan(api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d,
                                similarity=api.SIM_MSE, lambda_diff=0.0, diffeo_steps=2))
    print(f"case squaring forms {n}", flush=True)
    near_u = api.displacement(plan, gpu(th)).clone()
    far_u = api.displacement(plan, gpu(far)).clone()
    torch.cuda.synchronize()
    corner = (slice(None),) + (slice(0, 8),) * d
    assert not torch.equal(near_u[corner], far_u[corner])
    near_u[corner] = 0.0
    far_u[corner] = 0.0
    bad = (near_u != far_u).sum().item()
    assert bad == 0, f"{bad} of {near_u.numel()} differ"


# The adjoint of a squaring that moves less than one voxel sums a voxel's
# transposed terms in 64 bits. A constant displacement of eighths has exact
# weights, and the image gradient is zero at every second voxel, where the
# result is the transposed sum alone: rounded once, it lies within 2^-24 of its
# own size, also where its terms cancel (2^-23 asserted; 32-bit sums are off by
# 2^-24 of the largest term).
@pytest.mark.parametrize("n", [(65, 33, 17), (129, 65)])
def test_transposed_sums_in_64_bits(n):
    d = len(n)
    shape = tuple(reversed(n))
    disp = (3 / 8, -1 / 4, 1 / 8)[:d]
    th = np.zeros((d,) + shape)
    for a in range(d):
        th[a] = 2 * disp[a] * 2.0 / (n[a] - 1)     # u_0 = theta / 2; exact: n - 1 is a power of 2
    x = np.broadcast_to(np.arange(n[0], dtype=np.float64), shape)
    F = x + np.random.default_rng(3).normal(0.0, 8.0, shape)
    even = (np.arange(n[0]) % 2) == 0
    F[..., even] = (x + 2 * disp[0])[..., even]    # the warped image there, exactly
    one = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d, similarity=api.SIM_MSE,
                      lambda_diff=0.0, diffeo_steps=1)
    zero = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d, similarity=api.SIM_MSE,
                       lambda_diff=0.0, diffeo_steps=0)
    print(f"case transposed sums {n}", flush=True)
    p1 = api.Plan(one)
    u1 = api.displacement(p1, gpu(th))
    _, g1 = api.objective_and_grad(p1, gpu(F), gpu(x), gpu(th))
    _, g0 = api.objective_and_grad(api.Plan(zero), gpu(F), gpu(x), u1)
    g = g0[0].double().cpu().numpy()               # dL/du_1 along x
    want = np.zeros(shape)
    for c in range(2 ** d):
        w, moved = 1.0, g
        for a in range(d):
            fl = np.floor(disp[a])
            f = disp[a] - fl
            bit = (c >> a) & 1
            w *= f if bit else 1.0 - f
            moved = np.roll(moved, int(fl) + bit, axis=d - 1 - a)
        want += w * moved
    inner = (slice(3, -3),) * d
    got = 2.0 * g1[0].double().cpu().numpy()       # dL/du_0 = 2 dL/dtheta
    at = np.zeros(shape, bool)
    at[..., even] = True
    at, got, want, g = at[inner], got[inner], want[inner], g[inner]
    assert np.all(g[at] == 0.0) and np.all(want[at] != 0.0)
    err = np.max(np.abs(got[at] - want[at]) / np.abs(want[at]))
    print(f"largest relative error {err:.2e}", flush=True)
    assert err <= 2.0 ** -23


# The largest volumes but one: the lanes of a last, partial block of columns
# address their buffers past 4 N bytes, so nothing but its owner writes the
# last voxels. Constant images: the gradient is the total variation's, a sum of
# signs, and exact up to the rounding of its factor.
def test_largest_volume_last_voxels():
    n = (870, 4859, 127)                                     # 2^29 - 2 voxels
    lam = 0.5
    plan = api.Plan(api.Problem(n=n, transform=api.TF_DENSE, spacing=(1, 1, 1),
                                similarity=api.SIM_MSE, lambda_diff=lam,
                                regulariser=api.REG_ANISO_TV))
    print(f"case largest volume {n}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    F = torch.zeros(tuple(reversed(n)), device=DEV)
    th = torch.empty((3,) + tuple(reversed(n)), device=DEV)
    th.normal_(0.0, 1e-4, generator=gen)
    _, g = api.objective_and_grad(plan, F, F, th)
    u = th[:, -3:].double()                                  # the last three planes
    want = torch.zeros_like(u)
    inner = (slice(None),) + (slice(0, -1),) * 3             # the term's points
    for a in range(3):
        ahead = [slice(None)] + [slice(0, -1)] * 3
        ahead[1 + a] = slice(1, None)
        k = torch.sign(u[tuple(ahead)] - u[inner])
        want[tuple(ahead)] += k
        want[inner] -= k
    want *= lam / ((n[0] - 1) * (n[1] - 1) * (n[2] - 1))
    got = g[:, -2:].double()
    err = (got - want[:, -2:]).abs().max().item() / want.abs().max().item()
    print(f"largest error {err:.2e}", flush=True)
    assert err <= 1e-6


def inputs(n, seed):
    rng = np.random.default_rng(seed)
    shape = tuple(reversed(n))
    F = synth.blobs(shape, 10, rng) + rng.normal(0, 0.01, shape)
    M = synth.blobs(shape, 10, rng) + rng.normal(0, 0.01, shape)
    return F.astype(np.float32), (0.5 * M + 0.5 * F).astype(np.float32)


def unused_voxels(n, u):
    """Masks of the voxels whose sample point lies outside the volume and of
    the moving image's voxels that no point inside reads; points within 1e-3
    voxel of a decision count as inside, and as reading both cells."""
    d = len(n)
    out = np.zeros(tuple(reversed(n)), bool)
    pts = []
    for a in range(d):
        x = np.arange(n[a], dtype=np.float64).reshape((-1,) + (1,) * a)
        with np.errstate(invalid="ignore"):
            p = x + u[a].astype(np.float64) * (n[a] - 1) / 2
            out |= ~((p >= -1e-3) & (p <= n[a] - 1 + 1e-3))
        pts.append(p)
    read = np.zeros(tuple(reversed(n)), bool)
    inside = [p[~out] for p in pts]
    for c in range(4 ** d):                   # floor(p - 1e-3), floor(p + 1e-3), and the next ones
        idx = []
        for a in range(d):
            k = (c >> (2 * a)) & 3
            j = np.floor(inside[a] + (1e-3 if k & 1 else -1e-3)).astype(np.int64) + (k >> 1)
            idx.append(np.clip(j, 0, n[a] - 1))
        read[tuple(reversed(idx))] = True
    return out, ~read


# What lies outside the mask does not count, whatever it holds: NaN and
# infinities in the fixed image there and in the moving image where no sample
# inside reads, and displacements so large that the sample overflows. 16 x 16
# and other tiles, odd and even cells, and a grid too fine for the pipelined
# kernel.
@pytest.mark.parametrize("n,sp,tiling", [((45, 38, 41), (10, 10, 10), None),
                                         ((45, 38, 41), (5, 5, 5), None),
                                         ((70, 37, 44), (6, 7, 5), 2), ((70, 37, 44), (6, 7, 5), 3),
                                         ((40, 36, 33), (20, 16, 33), None),
                                         ((40, 24, 33), (3, 1, 6), None)])
@pytest.mark.parametrize("sim", [api.SIM_MSE, api.SIM_NCC])
def test_non_finite_outside_the_mask_3d(n, sp, tiling, sim):
    check_non_finite_outside(n, sp, sim, tiling)


def check_non_finite_outside(n, sp, sim, tiling=None):
    d = len(n)
    kw = dict(n=n, spacing=sp, similarity=sim, lambda_diff=0.0)
    p = api.Problem(**kw)
    F, M = inputs(n, 31)
    th = synth.random_theta(n, sp, 4.0, 32)
    th[(slice(None),) + (-1,) * d] = 1e25
    th[(slice(None),) + (-2,) * d] = -1e30
    print(f"case non-finite outside {n} {sp} sim={sim} tiling={tiling}", flush=True)
    plan = api.Plan(p) if tiling is None else api.Plan(p, tiling=tiling)
    u = api.displacement(plan, gpu(th)).cpu().numpy()
    out, unread = unused_voxels(n, u)
    assert out.sum() > 50 and unread.sum() > 50
    vo, go, _ = O.objective_and_grad(O.Problem(**kw), F, M, th)
    assert np.isfinite(vo) and np.all(np.isfinite(go))
    rng = np.random.default_rng(33)
    bad = np.array([np.nan, np.inf, -np.inf], np.float32)
    Fb, Mb = F.copy(), M.copy()
    Fb[out] = bad[rng.integers(0, 3, int(out.sum()))]
    Mb[unread] = bad[rng.integers(0, 3, int(unread.sum()))]
    v, g = api.objective_and_grad(plan, gpu(Fb), gpu(Mb), gpu(th))
    assert api.get_flags(plan) == [0]
    assert abs(float(v) - vo) <= VAL_TOL * abs(vo), (float(v), vo)
    check_grad(g.double().cpu().numpy(), go, f"non-finite outside {n} {sp}")


# the same in 2D: one block per small pair, and tiles (whose NCC shift may come
# from a voxel outside the mask too)
@pytest.mark.parametrize("n,sp,tiles", [((64, 64), (8, 8), False), ((64, 64), (8, 8), True),
                                        ((41, 50), (4, 5), False), ((41, 50), (4, 5), True),
                                        ((150, 131), (16, 16), False)])
@pytest.mark.parametrize("sim", [api.SIM_MSE, api.SIM_NCC])
def test_non_finite_outside_the_mask_2d(n, sp, tiles, sim):
    p = api.Problem(n=n, spacing=sp, similarity=sim, lambda_diff=0.0)
    check_non_finite_outside(n, sp, sim, api.Plan(p).tiling if tiles else None)


def test_non_finite_image_centre_outside_the_mask():
    """The voxel that the one-block kernel takes its NCC shift from lies
    outside the mask and holds a NaN."""
    n = (48, 40)
    kw = dict(n=n, spacing=(8, 8), similarity=api.SIM_NCC, lambda_diff=0.0)
    F, M = inputs(n, 41)
    nc = api.Problem(**kw).ncontrol()
    th = np.zeros((2, nc[1], nc[0]), np.float32)
    # the middle columns leave the image; no sample lands on a voxel, where the
    # gradient jumps (a sixth of the displacement is no whole number)
    th[0, :, 3:6] = 61.3 * 2.0 / (n[0] - 1)
    plan = api.Plan(api.Problem(**kw))
    out, _ = unused_voxels(n, api.displacement(plan, gpu(th)).cpu().numpy())
    c = (n[1] // 2, n[0] // 2)
    assert out[c] and not out.all()
    vo, go, _ = O.objective_and_grad(O.Problem(**kw), F, M, th)
    F[c] = np.nan
    print("case centre", flush=True)
    v, g = api.objective_and_grad(plan, gpu(F), gpu(M), gpu(th))
    assert abs(float(v) - vo) <= VAL_TOL * abs(vo), (float(v), vo)
    check_grad(g.double().cpu().numpy(), go, "centre")


# The one-block kernel sums a control's support in 64 bits. No displacement, a
# ramp for the moving image and differences that are exact in FP32: each pixel's
# term is known, and a control's value is off by the rounding of its columns'
# sums (2^-24 of each) and of the result. The rows' terms nearly cancel, so a
# 32-bit sum is off by 2^-24 of the much larger terms.
@pytest.mark.parametrize("n,sp", [((64, 64), 8), ((48, 51), 16), ((100, 40), 12)])
def test_small_2d_sums_in_64_bits(n, sp):
    shape = tuple(reversed(n))
    rng = np.random.default_rng(51)
    x = np.broadcast_to(np.arange(n[0], dtype=np.float64), shape)
    sign = np.where(np.arange(n[1]) % 2 == 0, 1.0, -1.0)[:, None]
    r = sign * 2000.0 + rng.integers(-1023, 1024, shape) / 1024.0
    F = x - r                                        # exact: 23 bits
    assert np.all(F.astype(np.float32) == F)
    p = api.Problem(n=n, spacing=(sp, sp), similarity=api.SIM_MSE, lambda_diff=0.0)
    plan = api.Plan(p)
    nc = p.ncontrol()
    print(f"case 64-bit sums {n} {sp}", flush=True)
    _, g = api.objective_and_grad(plan, gpu(F), gpu(x), gpu(np.zeros((2, nc[1], nc[0]))))
    got = g[0].double().cpu().numpy()

    def weights(m, c):                               # [c][m], the FP32 weights
        w = np.zeros((c, m))
        for v in range(m):
            t = (v % sp) / sp
            b = [(1 - t) ** 3 / 6, (3 * t ** 3 - 6 * t * t + 4) / 6,
                 (-3 * t ** 3 + 3 * t * t + 3 * t + 1) / 6, t ** 3 / 6]
            w[v // sp:v // sp + 4, v] = np.float32(b)
        return w

    wx, wy = weights(n[0], nc[0]), weights(n[1], nc[1])
    dx = np.ones(shape)
    dx[:, -1] = -(n[0] - 1)                          # right of the last voxel is zero
    cols = wy @ (r * dx).astype(np.float32).astype(np.float64)   # FP32 terms
    want = cols @ wx.T
    scale = 2.0 / (n[0] * n[1]) * (n[0] - 1) / 2
    bound = scale * (2.0 ** -24 * (np.abs(cols) @ wx.T) + 2.0 ** -23 * np.abs(want))
    worst = np.max(np.abs(got - scale * want) / bound)
    print(f"largest error over its bound {worst:.2f}", flush=True)
    assert worst <= 1.0


# The last batch of one block per pair and the first on tiles, the largest pairs
# of either size class and one pixel row more, the longest side, the most
# control rows.
@pytest.mark.parametrize("n,sp,pairs", [((32, 32), 8, 512), ((32, 32), 8, 513),
                                        ((64, 64), 8, 1), ((64, 65), 8, 1), ((64, 112), 12, 1),
                                        ((64, 113), 12, 1), ((80, 80), 16, 256),
                                        ((80, 80), 16, 257), ((256, 16), 16, 1), ((257, 15), 16, 1),
                                        ((64, 57), 2, 1), ((64, 59), 2, 1)])
def test_one_block_or_tiles(n, sp, pairs):
    kw = dict(n=n, spacing=(sp, sp), similarity=api.SIM_NCC, lambda_diff=0.1)
    data = [inputs(n, 60 + i) for i in range(3)]
    ths = [synth.random_theta(n, (sp, sp), 0.8, 70 + i) for i in range(3)]
    pick = [0] * pairs
    pick[pairs // 2], pick[-1] = 1, 2
    dev = [tuple(gpu(a) for a in (f, m, t)) for (f, m), t in zip(data, ths)]
    print(f"case one block or tiles {n} {sp} x {pairs}", flush=True)
    vals, grads, _ = api.objective_and_grad_batched(
        api.Plan([api.Problem(**kw)] * pairs), *([dev[k][j] for k in pick] for j in range(3)))
    for i in sorted({0, pairs // 2, pairs - 1}):
        vo, go, _ = O.objective_and_grad(O.Problem(**kw), *data[pick[i]], ths[pick[i]])
        assert abs(float(vals[i]) - vo) <= VAL_TOL * abs(vo)
        check_grad(grads[i].double().cpu().numpy(), go, f"pair {i} of {pairs}")


# The edges of the linear convolution form's rule: its channels (1.5 channel
# tiles, no vector epilogue, 16 channels in), the longest rows of 128-, 64- and
# 32-voxel blocks and one more, the smallest launch of 128-voxel blocks and one
# less, a round of blocks and a second one too short.
@pytest.mark.parametrize("cin,cout,dims,batch", [
    (24, 24, (33, 29, 27), 1), (32, 20, (40, 40, 17), 1), (16, 48, (33, 33, 46), 1),
    (16, 80, (33, 33, 46), 1), (48, 32, (75, 19, 18), 1), (48, 32, (76, 19, 18), 1),
    (64, 32, (55, 15, 14), 1), (64, 32, (56, 15, 14), 1), (96, 48, (67, 5, 6), 1),
    (96, 48, (68, 5, 6), 1), (32, 16, (25, 32, 32), 1), (32, 16, (25, 31, 33), 1),
    (32, 16, (31, 31, 34), 1), (32, 16, (31, 32, 34), 1)])
def test_conv_form_edges(cin, cout, dims, batch):
    check_conv(cin, cout, dims, batch)


# The edges of the cell contractions' rules: coarse grids of few and of enough
# 16-cell groups, the most phases that go one by one and the next, and both in
# one plan (a volume past the expansion's limit is compared below).
@pytest.mark.parametrize("n,sp", [((50, 47, 49), (16, 16, 16)), ((48, 192, 176), (16, 16, 16)),
                                  ((48, 40, 30), (12, 12, 12)), ((60, 44, 40), (16, 12, 12)),
                                  ((42, 31, 30), (10, 10, 10)), ((45, 31, 30), (11, 10, 10))])
@pytest.mark.parametrize("kind", ["tv", "wendland"])
def test_contraction_form_edges(n, sp, kind):
    check_contraction(n, sp, kind)


def test_contraction_past_the_voxel_limit():
    """Phases along x that are no multiple of 4: the expansion by the general
    kernel (2^22 voxels and more) gives the bits of the other one, row by row."""
    sp = (10, 9, 7)
    us = []
    rng = np.random.default_rng(91)
    th = None
    for nz in (150, 126):                  # 4.33 and 3.64 million voxels, both sides of 2^22
        n = (170, 170, nz)
        p = api.Problem(n=n, spacing=sp, similarity=api.SIM_LCC, lambda_diff=0.1, lcc_radius=1)
        nc = p.ncontrol()
        if th is None:
            th = rng.normal(0.0, 0.01, (3, nc[2], nc[1], nc[0])).astype(np.float32)
        us.append(api.displacement(api.Plan(p), gpu(th[:, :nc[2]])))
    print("case expansion past the voxel limit", flush=True)
    assert torch.equal(us[0][:, :126], us[1])


# A dense gradient may be written over its parameters (and the images): the
# kernels that write it still read them.
@pytest.mark.parametrize("kw", [dict(similarity=api.SIM_MSE, diffeo_steps=3),
                                dict(similarity=api.SIM_NCC, diffeo_steps=1),
                                dict(similarity=api.SIM_LCC, lcc_radius=2),
                                dict(similarity=api.SIM_LCC, lcc_radius=2, diffeo_steps=2),
                                dict(similarity=api.SIM_LCC, lcc_radius=2,
                                     regulariser=api.REG_ISO_TV)])
@pytest.mark.parametrize("n", [(70, 40, 33), (130, 90)])
def test_dense_gradient_over_its_inputs(n, kw):
    d = len(n)
    p = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d, lambda_diff=0.2, **kw)
    F, M = inputs(n, 95)
    th = synth.smooth_dense(n, 1.0, 96)
    print(f"case gradient over its inputs {n} {kw}", flush=True)
    plan = api.Plan(p)
    v, g = api.objective_and_grad(plan, gpu(F), gpu(M), gpu(th))
    both = gpu(th)
    v2, g2 = api.objective_and_grad(plan, gpu(F), gpu(M), both, grad=both)
    assert torch.equal(v, v2) and torch.equal(g, g2)
    # theta, then the images, in one array; the gradient ends inside the images
    N = int(np.prod(n))
    arr = torch.cat([gpu(th).flatten(), gpu(F).flatten(), gpu(M).flatten()])
    shape = tuple(reversed(n))
    out = arr[N + 8:N + 8 + d * N].view((d,) + shape)
    v3, g3 = api.objective_and_grad(plan, arr[d * N:(d + 1) * N].view(shape),
                                    arr[(d + 1) * N:].view(shape),
                                    arr[:d * N].view((d,) + shape), grad=out)
    assert torch.equal(v, v3) and torch.equal(g, g3)


def test_conv_more_channels_than_lds_sizes_hold():
    """Staged runs of more than 2^31 bytes: another form takes the layer. A few
    non-zero operands, small whole numbers, so the result is exact."""
    from paper_1806_09907_amd import cnn
    nx, cin = 67, 2130448
    x = torch.zeros((nx, cin), dtype=torch.bfloat16, device=DEV)
    w = torch.zeros((1, 27 * cin), dtype=torch.bfloat16, device=DEV)
    want = np.zeros(nx)
    for v, c, val in [(0, 0, 2.0), (10, cin - 1, 3.0), (33, 1000003, -1.0), (66, 8, 5.0)]:
        x[v, c] = val
        for dx in range(3):
            w[0, (9 + 3 + dx) * cin + c] = dx + 1
            if 0 <= v + 1 - dx < nx:
                want[v + 1 - dx] += val * (dx + 1)
    y = torch.empty((nx, 1), dtype=torch.float32, device=DEV)
    print("case channels past the LDS sizes", flush=True)
    cnn.conv_fwd(x, (nx, 1, 1), cin, w, None, 1, 0, y_f32=y, batch=1)
    assert np.array_equal(y.double().cpu().numpy().ravel(), want)


# The one-block kernel and the autotuner: a call that fails leaves the plan on
# it, a call that finds it fastest keeps it, and the cache brings it back. The
# forms differ in their last bits, which tells them apart.
def test_autotune_knows_the_one_block_kernel(tmp_path):
    n, sp = (64, 61), (8, 8)
    F, M = inputs(n, 97)
    th = synth.random_theta(n, sp, 0.8, 98)
    args = [gpu(F)], [gpu(M)], [gpu(th)]
    prob = api.Problem(n=n, spacing=sp, similarity=api.SIM_NCC, lambda_diff=0.05)

    def grad(plan):
        return api.objective_and_grad(plan, args[0][0], args[1][0], args[2][0])[1]

    plan = api.Plan(prob)
    whole = grad(plan)
    tiles = grad(api.Plan(prob, tiling=plan.tiling))
    assert not torch.equal(whole, tiles)
    print("case autotune, workspace too small", flush=True)
    out = torch.empty_like(args[2][0])
    table = api.PointerTable(*args, [out], DEV)
    values = torch.empty(1, device=DEV)
    chosen, ms = ctypes.c_int32(-1), ctypes.c_double(0.0)
    st = lib().air_autotune(plan.handle, api._ptr(table.fixed), api._ptr(table.moving),
                            api._ptr(table.theta), api._ptr(values), api._ptr(table.grads), None, 0,
                            2, None, ctypes.byref(chosen), ctypes.byref(ms), api._stream())
    assert st != 0
    assert torch.equal(grad(plan), whole)
    print("case autotune", flush=True)
    cache = str(tmp_path / "tune.json")
    rep = tune.autotune(plan, *args, reps=20, cache_path=cache)
    assert rep["tiling"] == plan.tiling
    assert torch.equal(grad(plan), whole)
    fresh = api.Plan(prob)
    assert tune.cached_tiling(fresh, cache) == rep["tiling"]
    assert torch.equal(grad(fresh), whole)
    # a caller's choice of tiles stays one
    tiled = api.Plan(prob, tiling=rep["tiling"])
    assert torch.equal(grad(tiled), tiles)


# The mask is decided on the exact point: a displacement far below the rounding
# of the point itself puts the last voxels of an axis outside (positive) or
# leaves them inside (negative), the first ones the other way round.
@pytest.mark.parametrize("n,sp", [((33, 21, 30), 10), ((33, 21, 30), 5), ((40, 36, 33), 16),
                                  ((40, 24, 33), (3, 1, 6)), ((50, 41), 8), ((150, 131), 12)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_mask_a_hair_past_the_last_voxel(n, sp, sign):
    d = len(n)
    sp = (sp,) * d if isinstance(sp, int) else sp
    kw = dict(n=n, spacing=sp, similarity=api.SIM_MSE, lambda_diff=0.0)
    p = api.Problem(**kw)
    F, M = inputs(n, 101)
    plan = api.Plan(p)
    for a in range(d):
        th = np.zeros(p.param_shape(), np.float32)
        th[a] = sign * 3e-8 * 2.0 / (n[a] - 1)
        print(f"case hair {n} {sp} axis {a} sign {sign}", flush=True)
        v, _ = api.objective_and_grad(plan, gpu(F), gpu(M), gpu(th))
        vo, _, _ = O.objective_and_grad(O.Problem(**kw), F, M, th)
        assert abs(float(v) - vo) <= VAL_TOL * abs(vo), (a, float(v), vo)
