"""Objective and gradient against the FP64 oracle at the sizes where the
kernels' work splits change: remainders of a block's walk, the shortest and
longest walks, tile edges. Tolerances are the parity bars of every GPU test
(parity.py): 1e-5 for the value, 1e-4 for the gradient (norm- and
element-wise)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1806_09907_amd import api, synth
from paper_1806_09907_amd._lib import AirError
from parity import VAL_TOL, check_grad

pytestmark = pytest.mark.gpu
DEV = "cuda"


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def inputs(n, seed, blobs=10):
    rng = np.random.default_rng(seed)
    F = synth.blobs(tuple(reversed(n)), blobs, rng) + rng.normal(0, 0.01, tuple(reversed(n)))
    M = synth.blobs(tuple(reversed(n)), blobs, rng) + rng.normal(0, 0.01, tuple(reversed(n)))
    return F.astype(np.float32), (0.5 * M + 0.5 * F).astype(np.float32)


def check(p, F, M, th, what):
    print(f"case {what}", flush=True)
    plan = api.Plan(p)
    v, g = api.objective_and_grad(plan, gpu(F), gpu(M), gpu(th))
    torch.cuda.synchronize()
    op = O.Problem(n=p.n, transform=p.transform, spacing=p.spacing, similarity=p.similarity,
                   lambda_diff=p.lambda_diff, diffeo_steps=p.diffeo_steps,
                   regulariser=p.regulariser, sigma=p.sigma, lcc_radius=p.lcc_radius)
    vo, go, _ = O.objective_and_grad(op, F, M, th)
    assert abs(float(v) - vo) <= VAL_TOL * abs(vo), (float(v), vo)
    check_grad(g.double().cpu().numpy(), go, what)


# dense passes: walks of 8, 16 and 32 planes (1, 2, .. 8 row groups in 2D) and
# their remainders
@pytest.mark.parametrize("n", [(70, 9, 7), (66, 5, 8), (64, 4, 9), (65, 6, 17), (256, 256, 150),
                               (256, 256, 254), (64, 3), (65, 301), (700, 1100)])
@pytest.mark.parametrize("sim", [api.SIM_MSE, api.SIM_NCC])
def test_dense_walks(n, sim):
    p = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * len(n), similarity=sim,
                    lambda_diff=0.5)
    F, M = inputs(n, 7)
    rng = np.random.default_rng(8)
    th = rng.normal(0.0, 1.5, (len(n),) + tuple(reversed(n)))
    for a in range(len(n)):
        th[a] *= 2.0 / (n[a] - 1)
    check(p, F, M, th.astype(np.float32), f"dense walk {n} sim={sim}")


def test_dense_batch_uneven_walks():
    """Pairs of one batch share the walk length; each keeps its own blocks."""
    sizes = [(33, 12, 9), (70, 5, 31), (64, 8, 8)]
    probs = [api.Problem(n=n, transform=api.TF_DENSE, spacing=(1, 1, 1), similarity=api.SIM_NCC,
                         lambda_diff=0.2) for n in sizes]
    data = [inputs(n, 20 + i) for i, n in enumerate(sizes)]
    ths = [synth.random_dense(n, 1.0, 30 + i) for i, n in enumerate(sizes)]
    vals, grads, _ = api.objective_and_grad_batched(
        api.Plan(probs), [gpu(f) for f, _ in data], [gpu(m) for _, m in data],
        [gpu(t) for t in ths])
    torch.cuda.synchronize()
    for i, n in enumerate(sizes):
        op = O.Problem(n=n, transform=O.TF_DENSE, spacing=(1, 1, 1), similarity=O.SIM_NCC,
                       lambda_diff=0.2)
        vo, go, _ = O.objective_and_grad(op, data[i][0], data[i][1], ths[i])
        assert abs(float(vals[i]) - vo) <= VAL_TOL * abs(vo)
        check_grad(grads[i].double().cpu().numpy(), go, f"dense batch pair {i}")


# the exponential: near squarings (samples within one voxel, LDS ring), far
# ones, the first squaring's samples that leave the ring, walk and tile edges
@pytest.mark.parametrize("n,std,K", [((33, 9, 17), 1.5, 4), ((32, 8, 8), 1.5, 3),
                                     ((31, 7, 33), 3.0, 2), ((65, 10, 9), 4.0, 1),
                                     ((40, 24, 40), 6.0, 3), ((257, 9), 1.5, 4), ((255, 33), 6.0, 2),
                                     ((256, 64), 3.0, 3)])
@pytest.mark.parametrize("tf", [api.TF_DENSE, api.TF_BSPLINE3])
def test_exponential_walks(n, std, K, tf):
    d = len(n)
    sp = (1,) * d if tf == api.TF_DENSE else (5,) * d
    p = api.Problem(n=n, transform=tf, spacing=sp, similarity=api.SIM_MSE, lambda_diff=0.1,
                    diffeo_steps=K)
    F, M = inputs(n, 50)
    th = (synth.smooth_dense(n, std, 51) if tf == api.TF_DENSE
          else synth.random_theta(n, sp, std, 51))
    check(p, F, M, th, f"exponential {n} std={std} K={K} tf={tf}")


# the pipelined kernel of any spacing: odd and even layer counts of a cell,
# the last cell cut by the volume after 1 .. spacing layers, windows of up to
# 16 controls (the general kernel beyond), coarse grids whose controls gather
# from many tiles (32 and 64 lanes per control), and each tile shape
@pytest.mark.parametrize("n,sp", [((33, 17, 31), (10, 10, 10)), ((47, 35, 41), (5, 7, 3)),
                                  ((40, 36, 25), (2, 2, 2)), ((19, 18, 20), (1, 1, 1)),
                                  ((40, 24, 33), (3, 1, 6)), ((70, 66, 65), (32, 32, 32)),
                                  ((128, 40, 36), (64, 16, 16)), ((97, 80, 64), (12, 20, 9)),
                                  ((2, 3, 2), (4, 4, 4)), ((16, 16, 17), (16, 16, 16))])
@pytest.mark.parametrize("sim", [api.SIM_MSE, api.SIM_NCC])
def test_any_spacing(n, sp, sim):
    p = api.Problem(n=n, spacing=sp, similarity=sim, lambda_diff=0.05)
    F, M = inputs(n, 60)
    check(p, F, M, synth.random_theta(n, sp, 0.8, 61), f"spacing {sp} {n} sim={sim}")


@pytest.mark.parametrize("tiling", range(10))
@pytest.mark.parametrize("sp", [(6, 6, 6), (3, 3, 5)])
def test_any_spacing_tilings(tiling, sp):
    n = (70, 37, 44)
    p = api.Problem(n=n, spacing=sp, similarity=api.SIM_NCC, lambda_diff=0.05)
    F, M = inputs(n, 62)
    th = synth.random_theta(n, sp, 0.8, 63)
    print(f"case spacing {sp} tiling {tiling}", flush=True)
    try:
        plan = api.Plan(p, tiling=tiling)
    except AirError as e:      # more LDS than a block may have
        assert e.status == 5
        return
    v, g = api.objective_and_grad(plan, gpu(F), gpu(M), gpu(th))
    vo, go, _ = O.objective_and_grad(O.Problem(n=n, spacing=sp, similarity=O.SIM_NCC,
                                               lambda_diff=0.05), F, M, th)
    assert abs(float(v) - vo) <= VAL_TOL * abs(vo)
    check_grad(g.double().cpu().numpy(), go, f"spacing {sp} tiling {tiling}")


# per-cell contractions of fields on the voxel grid: four controls per axis
# with whole and partial 16-cell groups, rows that end inside four phases,
# spacings that are no multiple of 4, grids of too few cells (the general
# kernels), and more controls per axis (likewise)
@pytest.mark.parametrize("n,sp", [((128, 9, 17), (8, 8, 8)), ((133, 20, 12), (8, 5, 4)),
                                  ((35, 33, 34), (6, 6, 6)), ((17, 16, 24), (8, 8, 8)),
                                  ((16, 24, 40), (8, 8, 8)), ((70, 13, 11), (4, 4, 4)),
                                  ((50, 21, 30), (10, 3, 7)), ((30, 12, 9), (1, 2, 3))])
@pytest.mark.parametrize("kind", ["tv", "lcc", "wendland", "wendland3"])
def test_field_contractions(n, sp, kind):
    kw = {}
    if kind.startswith("wendland"):
        kw = dict(transform=api.TF_WENDLAND,
                  sigma=tuple((2.0 if kind == "wendland" else 2.7) * s for s in sp))
    p = api.Problem(n=n, spacing=sp, similarity=api.SIM_LCC if kind == "lcc" else api.SIM_NCC,
                    lambda_diff=0.02, lcc_radius=2,
                    regulariser=api.REG_ISO_TV if kind == "tv" else api.REG_DIFFUSION, **kw)
    F, M = inputs(n, 70)
    th = synth.random_controls(n, p.ncontrol(), 0.7, 71)
    check(p, F, M, th, f"contraction {kind} {n} spacing {sp}")


# convolutions on linear blocks of 32, 64 and 128 voxels: partial last blocks,
# volume seams inside a block, channel counts that are no multiple of 8 or 16,
# and the weight gradient on rows padded to whole x blocks
@pytest.mark.parametrize("cin,cout,dims,batch", [
    (112, 48, (5, 3, 7), 3),       # 32-voxel blocks, several volumes per block
    (48, 64, (10, 9, 4), 2),       # 32
    (48, 32, (23, 24, 7), 3),      # 64
    (32, 48, (12, 15, 31), 3),     # 64; padded weight gradient with seams
    (8, 24, (33, 29, 27), 1),      # 128, 1.5 channel tiles
    (16, 20, (40, 40, 17), 1),     # 128, no vector epilogue
    (64, 128, (21, 16, 77), 1),    # 128, eight channel tiles, padded bank pitch
    (112, 16, (49, 30, 18), 1),    # rows too wide for the staged runs
])
def test_conv_linear_blocks(cin, cout, dims, batch):
    from paper_1806_09907_amd import cnn
    nx, ny, nz = dims
    rng = np.random.default_rng(cin + cout)

    def bf(a):
        return torch.from_numpy(np.asarray(a, np.float32)).to(DEV).bfloat16().contiguous()

    def host(t):
        return t.double().cpu().numpy()

    x = bf(rng.normal(size=(batch * nz, ny, nx, cin)))
    w = bf(rng.normal(size=(cout, 27 * cin)) / np.sqrt(27 * cin))
    gate = bf(rng.normal(size=(batch * nz, ny, nx, cout)))
    b = rng.normal(size=cout).astype(np.float32)
    shape = (batch * nz, ny, nx, cout)
    y = torch.empty(shape, dtype=torch.float32, device=DEV)
    yb = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    print(f"case conv {cin}->{cout} {dims} x {batch}", flush=True)
    cnn.conv_fwd(x, dims, cin, w, gpu(b), cout, 1, y_bf=yb, y_f32=y, batch=batch)
    yg = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    cnn.conv_fwd(x, dims, cin, w, None, cout, 2, y_bf=yg, batch=batch, gate=gate, ldg=cout)
    xh, wh, gh = host(x), host(w), host(gate)
    pre = np.concatenate([O.conv3d_fwd(xh[v * nz:(v + 1) * nz], wh) for v in range(batch)])
    ref = pre + b.astype(np.float64)
    ref = np.where(ref > 0, ref, 0.1 * ref)
    assert np.linalg.norm(host(y) - ref) <= 1e-5 * np.linalg.norm(ref)
    assert torch.equal(yb, y.bfloat16())
    refg = np.where(gh > 0, pre, 0.1 * pre)
    # one rounding to bf16 on top: half an ulp, 2^-9 of each value
    assert np.all(np.abs(host(yg) - refg) <= 2.0 ** -8 * np.abs(refg) + 1e-4)
    if cout % 8 == 0:
        dy = bf(rng.normal(size=shape))
        dw = torch.empty((cout, 27 * cin), dtype=torch.float32, device=DEV)
        db = torch.empty(cout, dtype=torch.float32, device=DEV)
        cnn.conv_bwd_weight(x, dims, cin, dy, cout, dw, db, cnn.Workspace(DEV), batch=batch)
        dyh = host(dy)
        rw, rb = np.zeros((cout, 27 * cin)), np.zeros(cout)
        for v in range(batch):
            _, dwv, dbv = O.conv3d_bwd(xh[v * nz:(v + 1) * nz], wh, dyh[v * nz:(v + 1) * nz])
            rw, rb = rw + dwv, rb + dbv
        assert np.linalg.norm(host(dw) - rw) <= 1e-5 * np.linalg.norm(rw)
        assert np.linalg.norm(host(db) - rb) <= 1e-5 * np.linalg.norm(rb)


# small 2D pairs, one block each: the edges of 1, 2, 4 and 7 pixels per thread,
# controls as dense as the pixels, one cell for the whole image, the last
# size before the tiles, and images no wider than a cell
SMALL2 = [((32, 32), (8, 8)), ((33, 31), (8, 8)), ((64, 32), (5, 3)), ((41, 50), (4, 4)),
          ((64, 64), (8, 8)), ((65, 63), (8, 16)), ((112, 64), (8, 8)), ((7168 // 2, 2), (16, 1)),
          ((2, 2), (4, 4)), ((9, 300), (2, 64)), ((40, 41), (1, 1)), ((3, 1000), (8, 8))]


@pytest.mark.parametrize("n,sp", SMALL2)
@pytest.mark.parametrize("sim", [api.SIM_MSE, api.SIM_NCC])
def test_small_2d_one_block(n, sp, sim):
    p = api.Problem(n=n, spacing=sp, similarity=sim, lambda_diff=0.1)
    F, M = inputs(n, 80)
    check(p, F, M, synth.random_theta(n, sp, 0.8, 81), f"small 2D {n} spacing {sp} sim={sim}")


def test_small_2d_batch_flags_and_tiles():
    """A batch of small pairs; one of them entirely outside (degenerate), one
    with a NaN control (non-finite); and the tiles a caller selects agree."""
    sizes = [(40, 31), (64, 64), (33, 70), (20, 20)]
    probs = [api.Problem(n=n, spacing=(8, 8), similarity=api.SIM_NCC, lambda_diff=0.05)
             for n in sizes]
    data = [inputs(n, 90 + i) for i, n in enumerate(sizes)]
    ths = [synth.random_theta(n, (8, 8), 1.0, 95 + i) for i, n in enumerate(sizes)]
    ths[2] = ths[2] + np.float32(5.0)
    ths[3] = ths[3].copy()
    ths[3][0, 2, 2] = np.nan
    F, M, T = ([gpu(d[0]) for d in data], [gpu(d[1]) for d in data], [gpu(t) for t in ths])
    plan = api.Plan(probs)
    vals, grads, _ = api.objective_and_grad_batched(plan, F, M, T)
    flags = api.get_flags(plan)
    assert flags[0] == flags[1] == 0
    assert flags[2] == api.FLAG_DEGENERATE and flags[3] & api.FLAG_NONFINITE
    tiled = api.Plan(probs, tiling=plan.tiling)
    vt, gt, _ = api.objective_and_grad_batched(tiled, F, M, T)
    assert api.get_flags(tiled) == flags
    for i in range(3):
        if i == 2:
            assert torch.equal(grads[i], gt[i])
            continue
        op = O.Problem(n=sizes[i], spacing=(8, 8), similarity=O.SIM_NCC, lambda_diff=0.05)
        vo, go, _ = O.objective_and_grad(op, data[i][0], data[i][1], ths[i])
        for v, g in ((vals, grads), (vt, gt)):
            assert abs(float(v[i]) - vo) <= VAL_TOL * abs(vo)
            check_grad(g[i].double().cpu().numpy(), go, f"small 2D batch pair {i}")


# LCC: tiles of 32 x 8 columns and their remainders, one to several z chunks
# (shorter than the window too), every radius of the fused passes and one past
# them, samples outside the volume
@pytest.mark.parametrize("n,r", [((33, 9, 5), 1), ((31, 8, 3), 4), ((64, 17, 70), 3),
                                 ((100, 40, 9), 2), ((32, 16, 37), 4), ((34, 7, 12), 5)])
@pytest.mark.parametrize("tf", [api.TF_DENSE, api.TF_BSPLINE3])
def test_lcc_walks(n, r, tf):
    p = api.Problem(n=n, transform=tf, spacing=(1, 1, 1) if tf == api.TF_DENSE else (8, 8, 8),
                    similarity=api.SIM_LCC, lcc_radius=r, lambda_diff=0.1)
    F, M = inputs(n, 17)
    shape = (3,) + tuple(reversed(n)) if tf == api.TF_DENSE else p.param_shape()
    th = np.random.default_rng(18).normal(0.0, 0.5, shape)
    for a in range(3):
        th[a] *= 2.0 / (n[a] - 1)
    check(p, F, M, th.astype(np.float32), f"lcc walk {n} r={r} tf={tf}")


@pytest.mark.parametrize("n", [(2, 9, 7), (5, 300, 4), (257, 3, 11), (70, 41), (3, 65)])
def test_lcc_sampling_far_outside(n):
    """Paired gathers at every kind of edge: displacements of up to more than
    half the volume. The window of radius 8 keeps every variance far from 0,
    where the coefficients are well conditioned."""
    d = len(n)
    p = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d, similarity=api.SIM_LCC,
                    lcc_radius=8, lambda_diff=0.0)
    F, M = inputs(n, 19, 6)
    th = np.random.default_rng(20).uniform(-1.2, 1.2, (d,) + tuple(reversed(n))).astype(np.float32)
    check(p, F, M, th, f"lcc outside {n}")


# total variation: walks of 1, 2, 4 and 8 planes with their remainders, columns
# that end inside a block, the thinnest volumes
@pytest.mark.parametrize("n", [(2, 2, 2), (33, 9, 5), (128, 70, 33), (130, 127, 31),
                               (129, 128, 57), (200, 180, 41), (300, 2), (65, 70)])
@pytest.mark.parametrize("reg", [api.REG_ANISO_TV, api.REG_ISO_TV])
def test_tv_walks(n, reg):
    d = len(n)
    p = api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d, similarity=api.SIM_MSE,
                    lambda_diff=0.3, regulariser=reg)
    F, M = inputs(n, 21)
    th = np.random.default_rng(22).normal(0.0, 1.0, (d,) + tuple(reversed(n)))
    for a in range(d):
        th[a] *= 2.0 / (n[a] - 1)
    check(p, F, M, th.astype(np.float32), f"tv walk {n} reg={reg}")
