"""Measured cases of the registration framework.

Each case is one call (or one layer's calls) that a registration program
makes over and over: the objective and its gradient for one pair or a batch
of pairs, over the transformations, similarities, regularisers and sizes the
framework has, and the three directions of one layer of the learned
initialisation. `listed()` holds typical and extreme sizes, `draw()` gives
further ones of the same families, `exact()` computes a case in 64 bits with
plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as tnf
from torch.utils.checkpoint import checkpoint

from paper_1806_09907_amd import api, cnn

DEV = "cuda"
SIMS = {"mse": api.SIM_MSE, "ncc": api.SIM_NCC, "lcc": api.SIM_LCC}
TFS = {"bspline": api.TF_BSPLINE3, "dense": api.TF_DENSE, "wendland": api.TF_WENDLAND}
REGS = {"diffusion": api.REG_DIFFUSION, "aniso_tv": api.REG_ANISO_TV, "iso_tv": api.REG_ISO_TV}
BATCH_SIDES = (96, 112, 128, 144, 160)
CNN_LAYERS = {"e2": (16, 32, 4), "e3": (32, 48, 8), "e4": (48, 64, 16), "d1": (112, 48, 8)}


def _pair(name, nx, ny, nz, transform, sim, reg="diffusion", lam=0.05, sx=8, sy=8, sz=8, sigma=0.0,
          steps=0, radius=2):
    return {"name": name, "kind": "pair", "nx": nx, "ny": ny, "nz": nz, "transform": transform,
            "sim": sim, "reg": reg, "lam": lam, "sx": sx, "sy": sy, "sz": sz, "sigma": sigma,
            "steps": steps, "radius": radius}


def listed():
    return [
        # the smallest problem: a 2D slice registered interactively; latency
        _pair("bspline2d_64_mse", 64, 64, 1, "bspline", "mse", lam=0.1),
        # a 2D radiograph-like image of odd size, control spacing not a power of two
        _pair("bspline2d_odd_ncc", 1021, 769, 1, "bspline", "ncc", sx=12, sy=12),
        # one volume at the usual size and spacing: a serving or tuning loop over one pair
        _pair("bspline3d_128_ncc", 128, 128, 128, "bspline", "ncc"),
        # one brain-sized volume, odd sides, spacing 10: the general-spacing route
        _pair("bspline3d_odd_s10", 181, 217, 181, "bspline", "ncc", sx=10, sy=10, sz=10),
        # a cohort of uneven pairs in one launch: throughput
        {"name": "bspline3d_batch48", "kind": "batch", "pairs": 48, "sizes_seed": 1809907,
         "sim": "ncc", "lam": 0.05},
        # the finest level of a dense multi-resolution CT registration
        _pair("dense3d_256_mse", 256, 256, 256, "dense", "mse", lam=1.0),
        # a dense level of odd size with NCC
        _pair("dense3d_odd_ncc", 149, 181, 127, "dense", "ncc", lam=1.0),
        # diffeomorphic dense registration: exponential by six squarings
        _pair("diffeo3d_256_mse", 256, 256, 256, "dense", "mse", lam=1.0, steps=6),
        # edge-preserving regularisation of a control grid
        _pair("tv3d_128_ncc", 128, 128, 128, "bspline", "ncc", reg="aniso_tv", lam=0.02),
        # compactly supported radial basis instead of the B-spline
        _pair("wendland3d_128_ncc", 128, 128, 128, "wendland", "ncc", sigma=16.0),
        # local NCC: images whose contrast varies over the volume
        _pair("lcc3d_128_r3", 128, 128, 128, "bspline", "lcc", radius=3),
        # the decoder layer of the learned initialisation, 8 pairs of 128^3:
        # forward, backward-data and backward-weight of one training step
        {"name": "conv_d1_128_b8", "kind": "conv", "layer": "d1", "n": 128, "batch": 8},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fam = rng.choice(["bspline2d", "bspline3d", "bspline3d_any", "batch", "dense3d", "dense2d",
                      "diffeo3d", "diffeo2d", "tv", "wendland", "lcc", "conv"])
    sim = rng.choice(["mse", "ncc"])
    if fam == "bspline2d":
        s = rng.choice([4, 6, 8, 8, 12, 16])
        c = _pair("", _logint(rng, 48, 2048), _logint(rng, 48, 2048), 1, "bspline", sim, sx=s, sy=s)
    elif fam == "bspline3d":
        n = [rng.randint(64, 224) for _ in range(3)]
        c = _pair("", n[0], n[1], n[2], "bspline", sim)
    elif fam == "bspline3d_any":
        n = [rng.randint(64, 224) for _ in range(3)]
        s = rng.choice([(4, 4, 4), (5, 5, 5), (6, 6, 6), (10, 10, 10), (12, 12, 12), (16, 16, 16),
                        (32, 32, 32), (10, 10, 5), (12, 12, 6), (16, 16, 8)])
        c = _pair("", n[0], n[1], n[2], "bspline", sim, sx=s[0], sy=s[1], sz=s[2])
    elif fam == "batch":
        return {"kind": "batch", "pairs": rng.randint(4, 48), "sizes_seed": rng.randint(0, 1 << 30),
                "sim": sim, "lam": 0.05}
    elif fam == "dense3d":
        n = [rng.randint(64, 256) for _ in range(3)]
        c = _pair("", n[0], n[1], n[2], "dense", sim, lam=1.0)
    elif fam == "dense2d":
        c = _pair("", _logint(rng, 64, 4096), _logint(rng, 64, 4096), 1, "dense", sim, lam=1.0)
    elif fam == "diffeo3d":
        n = [rng.randint(64, 240) for _ in range(3)]
        tf = rng.choice(["dense", "bspline"])
        c = _pair("", n[0], n[1], n[2], tf, sim, lam=1.0 if tf == "dense" else 0.05,
                  steps=rng.randint(4, 7))
    elif fam == "diffeo2d":
        c = _pair("", _logint(rng, 128, 4096), _logint(rng, 128, 4096), 1, "dense", sim, lam=1.0,
                  steps=rng.randint(4, 7))
    elif fam == "tv":
        n = [rng.randint(64, 208) for _ in range(3)]
        tf = rng.choice(["dense", "bspline"])
        c = _pair("", n[0], n[1], n[2], tf, sim, reg=rng.choice(["aniso_tv", "iso_tv"]), lam=0.02)
    elif fam == "wendland":
        n = [rng.randint(64, 208) for _ in range(3)]
        s = rng.choice([6, 8, 8, 10])
        c = _pair("", n[0], n[1], n[2], "wendland", sim, sx=s, sy=s, sz=s,
                  sigma=float(rng.choice([2 * s, 2 * s, s + s // 2])))
    elif fam == "lcc":
        n = [rng.randint(64, 176) for _ in range(3)]
        c = _pair("", n[0], n[1], n[2], rng.choice(["dense", "bspline"]), "lcc",
                  radius=rng.randint(1, 4))
    else:
        return {"kind": "conv", "layer": rng.choice(sorted(CNN_LAYERS)),
                "n": 16 * rng.randint(4, 10), "batch": rng.randint(1, 8)}
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _blobs(n, count, gen):
    """Sum of isotropic Gaussian blobs over the grid n = (x, y[, z])."""
    out = None
    amp = torch.rand(count, generator=gen, device=DEV)
    sg = 3.0 + 7.0 * torch.rand(count, generator=gen, device=DEV)
    prof = []
    for m in n:
        c = torch.rand(count, generator=gen, device=DEV) * (m - 1)
        x = torch.arange(m, device=DEV, dtype=torch.float32)
        prof.append(torch.exp(-0.5 * ((x[None] - c[:, None]) / sg[:, None]) ** 2))
    prof[0] = prof[0] * amp[:, None]
    for b in range(count):
        v = prof[0][b]
        for p in prof[1:]:
            v = p[b].reshape((-1,) + (1,) * v.dim()) * v[None]
        out = v if out is None else out.add_(v)
    return out


def _ellipsoids(n, gen):
    """CT-like volume: smooth-edged ellipsoids of -1000..1000 on a background of -1000."""
    r = torch.rand((16, 7), generator=gen, device=DEV).cpu().numpy()
    d = len(n)
    vol = torch.full(tuple(reversed(n)), -1000.0, device=DEV)
    for k in range(16):
        q = 0.0
        for a in range(d):
            half = (0.03 + 0.28 * r[k, 3 + a]) * max(n)
            x = (torch.arange(n[a], device=DEV, dtype=torch.float32) - float(r[k, a] * n[a])) / half
            q = q + (x * x).reshape((-1,) + (1,) * a)
        vol = torch.where(q <= 1.0, torch.full_like(vol, float(2000.0 * r[k, 6] - 1000.0)), vol)
    pool = tnf.avg_pool2d if d == 2 else tnf.avg_pool3d
    for _ in range(2):
        vol = pool(vol[None, None], 3, 1, 1, count_include_pad=False)[0, 0]
    return vol


def _smooth_field(n, step, std, gen):
    """Smooth random displacement [d][..] in normalised units, std in voxels."""
    d = len(n)
    shape = tuple(reversed(n))
    coarse = torch.randn((1, d) + tuple(m // step + 3 for m in shape), generator=gen, device=DEV)
    u = tnf.interpolate(coarse, size=shape, mode="bilinear" if d == 2 else "trilinear",
                        align_corners=True)
    pool = tnf.avg_pool2d if d == 2 else tnf.avg_pool3d
    u = pool(u, 5, 1, 2, count_include_pad=False)[0]
    for a in range(d):
        u[a] *= std / float(u[a].std()) * 2.0 / (n[a] - 1)
    return u.contiguous()


def _warped(img, u, n):
    """img sampled at x + u(x) (zero padding), with plain torch."""
    d = len(n)
    grid = torch.stack([u[a] + torch.linspace(-1.0, 1.0, n[a], device=DEV).reshape(
        (-1,) + (1,) * a) for a in range(d)], dim=-1)
    return tnf.grid_sample(img[None, None], grid[None], mode="bilinear", padding_mode="zeros",
                           align_corners=True)[0, 0].contiguous()


def _images(n, gen, ct):
    """Fixed and moving image: blobs with noise, or CT-like; the moving one is
    the fixed one warped by a smooth field of a few voxels."""
    if ct:
        fixed = _ellipsoids(n, gen)
    else:
        fixed = _blobs(n, 12 if len(n) == 2 else 40, gen)
        fixed = fixed + 0.01 * torch.randn(fixed.shape, generator=gen, device=DEV)
    return fixed.contiguous(), _warped(fixed, _smooth_field(n, 24, 1.5, gen), n)


def _size(case):
    return (case["nx"], case["ny"]) if case["nz"] == 1 else (case["nx"], case["ny"], case["nz"])


def _problem(case):
    n = _size(case)
    d = len(n)
    sg = (case["sigma"],) * d if case["transform"] == "wendland" else ()
    sp = (1,) * d if case["transform"] == "dense" else (case["sx"], case["sy"], case["sz"])[:d]
    return api.Problem(n=n, transform=TFS[case["transform"]], spacing=sp,
                       similarity=SIMS[case["sim"]], lambda_diff=case["lam"],
                       diffeo_steps=case["steps"], regulariser=REGS[case["reg"]], sigma=sg,
                       lcc_radius=case["radius"])


def _pair_inputs(p, seed):
    gen = _gen(seed)
    ct = p.transform == api.TF_DENSE and p.similarity == api.SIM_MSE and p.dim == 3
    F, M = _images(p.n, gen, ct)
    if p.transform == api.TF_DENSE:
        th = _smooth_field(p.n, 12, 2.0, gen)
    else:
        std = 1.5 if p.diffeo_steps else (0.7 if p.transform == api.TF_WENDLAND else 1.0)
        th = std * torch.randn(p.param_shape(), generator=gen, device=DEV)
        for a in range(p.dim):
            th[a] *= 2.0 / (p.n[a] - 1)
    return F, M, th.contiguous()


def _batch_problems(case):
    rng = np.random.default_rng(case["sizes_seed"])
    return [api.Problem(n=tuple(int(v) for v in rng.choice(BATCH_SIDES, size=3)),
                        similarity=SIMS[case["sim"]], lambda_diff=case["lam"])
            for _ in range(case["pairs"])]


def _conv_inputs(case, seed):
    """One layer's operands: BF16 activations [v][cin], weights, bias, the
    gradient of the layer's output and the stored activation the data
    gradient is gated with (here the layer's input itself)."""
    cin, cout, div = CNN_LAYERS[case["layer"]]
    g = case["n"] // div
    gen = _gen(seed)
    vox = case["batch"] * g ** 3
    x = torch.randn((vox, cin), generator=gen, device=DEV)
    x = torch.where(x > 0, x, 0.1 * x).bfloat16()
    w = torch.randn((cout, 27, cin), generator=gen, device=DEV) * math.sqrt(2.0 / (27 * cin))
    b = 0.1 * torch.randn((cout,), generator=gen, device=DEV)
    dy = 0.01 * torch.randn((vox, cout), generator=gen, device=DEV)
    return cin, cout, g, x, w.bfloat16(), b, dy.bfloat16()


def prepare(case, seed):
    if case["kind"] == "pair":
        p = _problem(case)
        F, M, th = _pair_inputs(p, seed)
        plan = api.Plan(p)
        plan.prepare()
        plan.workspace(th.device)
        return {"kind": "pair", "plan": plan, "F": F, "M": M, "theta": th,
                "value": torch.empty((), device=DEV), "grad": torch.empty_like(th)}
    if case["kind"] == "batch":
        probs = _batch_problems(case)
        plan = api.Plan(probs)
        plan.prepare()
        F, M, T, G = [], [], [], []
        for i, p in enumerate(probs):
            f, m, t = _pair_inputs(p, seed * 1009 + i)
            F.append(f)
            M.append(m)
            T.append(t)
            G.append(torch.empty_like(t))
        plan.workspace(T[0].device)
        return {"kind": "batch", "plan": plan, "F": F, "M": M, "theta": T,
                "table": api.PointerTable(F, M, T, G, T[0].device),
                "values": torch.empty(len(probs), device=DEV)}
    cin, cout, g, x, w, b, dy = _conv_inputs(case, seed)
    wf = w.flip(1).permute(2, 1, 0).reshape(cin, 27 * cout).contiguous()
    return {"kind": "conv", "cin": cin, "cout": cout, "dims": (g, g, g), "batch": case["batch"],
            "x": x, "w": w.reshape(cout, 27 * cin).contiguous(), "wf": wf, "b": b, "dy": dy,
            "y": torch.empty((x.shape[0], cout), dtype=torch.bfloat16, device=DEV),
            "dx": torch.empty((x.shape[0], cin), dtype=torch.bfloat16, device=DEV),
            "dw": torch.empty((cout, 27 * cin), device=DEV), "db": torch.empty(cout, device=DEV),
            "ws": cnn.Workspace(x.device)}


def run(s):
    if s["kind"] == "pair":
        return api.objective_and_grad(s["plan"], s["F"], s["M"], s["theta"], value=s["value"],
                                      grad=s["grad"])
    if s["kind"] == "batch":
        values, grads, _ = api.objective_and_grad_batched(s["plan"], s["F"], s["M"], s["theta"],
                                                          values=s["values"], table=s["table"])
        return values, grads
    cin, cout, dims, B = s["cin"], s["cout"], s["dims"], s["batch"]
    cnn.conv_fwd(s["x"], dims, cin, s["w"], s["b"], cout, 1, y_bf=s["y"], batch=B)
    cnn.conv_fwd(s["dy"], dims, cout, s["wf"], None, cin, 2, y_bf=s["dx"], batch=B, gate=s["x"],
                 ldg=cin)
    cnn.conv_bwd_weight(s["x"], dims, cin, s["dy"], cout, s["dw"], s["db"], s["ws"], batch=B)
    return s["y"], s["dx"], s["dw"], s["db"]


# -------------------------------------------------------------------- work
def _pair_work(p):
    """Inputs read once, the gradient written once; the arithmetic of the
    expansion, the interpolation with its derivatives, the similarity's
    moments and the transposed expansion, per voxel."""
    vox = math.prod(p.n)
    par = math.prod(p.param_shape())
    flops = 60.0 if p.dim == 3 else 30.0
    if p.transform == api.TF_BSPLINE3:
        flops += 48.0 if p.dim == 3 else 32.0
    elif p.transform == api.TF_WENDLAND:
        flops += 4 * p.dim * math.prod(math.ceil(2 * p.sigma[a] / p.spacing[a])
                                       for a in range(p.dim))
    else:
        flops += 20.0
    if p.similarity == api.SIM_LCC:
        flops += 9 * 6 + 40.0
    flops += p.diffeo_steps * (3 * p.dim * 2 ** (p.dim + 1) + 20)
    return 4 * (2 * vox + 2 * par), flops * vox


def work(case):
    if case["kind"] == "pair":
        b, f = _pair_work(_problem(case))
    elif case["kind"] == "batch":
        w = [_pair_work(p) for p in _batch_problems(case)]
        b, f = sum(x[0] for x in w), sum(x[1] for x in w)
    else:
        cin, cout, div = CNN_LAYERS[case["layer"]]
        vox = case["batch"] * (case["n"] // div) ** 3
        b = vox * 2 * (3 * cin + 3 * cout) + cin * cout * 27 * (2 + 2 + 4)
        f = 3 * 2.0 * 27 * cin * cout * vox
    return {"bytes": b, "flops": f}


# ----------------------------------------------------------- 64-bit results
def _cubic(n, s):
    """[n][nc] matrix of the cubic B-spline with control j at (j - 1) s."""
    x = torch.arange(n, device=DEV)
    t = (x % s).double() / s
    w = torch.stack([(1 - t) ** 3 / 6, (3 * t ** 3 - 6 * t ** 2 + 4) / 6,
                     (-3 * t ** 3 + 3 * t ** 2 + 3 * t + 1) / 6, t ** 3 / 6], dim=1)
    m = torch.zeros((n, (n - 1) // s + 4), dtype=torch.float64, device=DEV)
    m.scatter_(1, (x // s)[:, None] + torch.arange(4, device=DEV)[None], w)
    return m


def _along(t, mat, axis):
    """mat [n][k] applied along `axis` of t."""
    t = t.movedim(axis, -1)
    return (t.reshape(-1, t.shape[-1]) @ mat.t().contiguous()).reshape(
        t.shape[:-1] + (mat.shape[0],)).movedim(-1, axis)


def _wendland(theta, p):
    """Sum over the lattice of psi_{3,2}(|(x - c) / sigma|) theta, cell by cell."""
    d = p.dim
    sg, sp = [float(v) for v in p.sigma], p.spacing
    m = [math.ceil(sg[a] / sp[a]) - 1 for a in range(d)]
    K = [m[a] + math.ceil((sp[a] - 1 + sg[a]) / sp[a]) for a in range(d)]
    cells = [(p.n[a] - 1) // sp[a] + 1 for a in range(d)]
    pad = []
    for a in range(d):                       # tnf.pad: last dimension (x) first
        pad += [0, max(0, cells[a] - 1 + K[a] - theta.shape[d - a])]
    theta = tnf.pad(theta, pad)
    out = torch.zeros([d] + [v for a in reversed(range(d)) for v in (cells[a], sp[a])],
                      dtype=torch.float64, device=DEV)
    grids = torch.meshgrid(*[torch.arange(K[a]) for a in reversed(range(d))], indexing="ij")
    for q in torch.stack([g.reshape(-1) for g in grids], 1).tolist():   # (z, y, x)
        r2 = 0.0
        for a in range(d):
            x = (torch.arange(sp[a], device=DEV, dtype=torch.float64)
                 - (q[d - 1 - a] - m[a]) * sp[a]) / sg[a]
            r2 = r2 + (x * x).reshape((-1,) + (1,) * a)
        r = r2.sqrt()
        w = torch.clamp(1 - r, min=0) ** 6 * (3 + 18 * r + 35 * r * r) / 3
        t = theta[(slice(None),) + tuple(slice(q[i], q[i] + cells[d - 1 - i]) for i in range(d))]
        if d == 2:
            out = out + t[:, :, None, :, None] * w[None, None, :, None, :]
        else:
            out = out + t[:, :, None, :, None, :, None] * w[None, None, :, None, :, None, :]
    out = out.reshape([d] + [cells[a] * sp[a] for a in reversed(range(d))])
    return out[(slice(None),) + tuple(slice(0, p.n[a]) for a in reversed(range(d)))]


def _points(u, n):
    d = len(n)
    return [torch.arange(n[a], device=DEV, dtype=torch.float64).reshape((-1,) + (1,) * a)
            + u[a] * (n[a] - 1) / 2 for a in range(d)]


def _sample(vol, pts, n):
    """vol [c][..] at the points, linear, zero outside."""
    d = len(n)
    flat = vol.reshape(vol.shape[0], -1)
    lo = [torch.floor(v.detach()) for v in pts]
    fr = [v - w for v, w in zip(pts, lo)]
    out = 0.0
    for corner in range(2 ** d):
        w, idx, ok, stride = 1.0, 0, True, 1
        for a in range(d):
            bit = (corner >> a) & 1
            c = lo[a] + bit
            ok = ok & (c >= 0) & (c <= n[a] - 1)
            idx = idx + c.clamp(0, n[a] - 1).long() * stride
            stride *= n[a]
            w = w * (fr[a] if bit else 1 - fr[a])
        val = flat.index_select(1, idx.reshape(-1)).reshape((vol.shape[0],) + idx.shape)
        out = out + val * (w * ok)
    return out


def _box(t, r):
    for a in range(t.dim()):
        t = t.movedim(a, -1)
        p = tnf.pad(t, (r, r))
        t = sum(p[..., k:k + t.shape[-1]] for k in range(2 * r + 1)).movedim(-1, a)
    return t


def _exact_pair(p, F, M, theta):
    n, d = p.n, p.dim
    F, M = F.double(), M.double()
    th = theta.double().requires_grad_(True)
    if p.transform == api.TF_DENSE:
        u = th
    elif p.transform == api.TF_WENDLAND:
        u = _wendland(th, p)
    else:
        u = th
        for a in range(d):
            u = _along(u, _cubic(n[a], p.spacing[a]), d - a)
    if p.diffeo_steps:
        u = u / 2.0 ** p.diffeo_steps
        for _ in range(p.diffeo_steps):
            u = checkpoint(lambda v: v + _sample(v, _points(v, n), n), u, use_reentrant=False)
    pts = _points(u, n)
    mask = True
    for a in range(d):
        mask = mask & (pts[a].detach() >= 0) & (pts[a].detach() <= n[a] - 1)
    W = _sample(M[None], pts, n)[0]
    cnt = mask.sum()
    if p.similarity == api.SIM_MSE:
        S = (((W - F) ** 2) * mask).sum() / cnt
    elif p.similarity == api.SIM_NCC:
        fc = (F - (F * mask).sum() / cnt) * mask
        wc = (W - (W * mask).sum() / cnt) * mask
        S = -(fc * wc).sum() / torch.sqrt((fc * fc).sum() * (wc * wc).sum())
    else:
        mk = mask.double()
        nw = _box(mk, p.lcc_radius).clamp(min=1)
        mf, mw = _box(mk * F, p.lcc_radius) / nw, _box(mk * W, p.lcc_radius) / nw
        vf = _box(mk * F * F, p.lcc_radius) / nw - mf * mf
        vw = _box(mk * W * W, p.lcc_radius) / nw - mw * mw
        cv = _box(mk * F * W, p.lcc_radius) / nw - mf * mw
        S = -(cv / torch.sqrt(vf * vw + 1e-10) * mk).sum() / cnt
    inner = (slice(None),) + tuple(slice(0, m - 1) for m in reversed(n))
    D = []
    for a in range(d):
        ahead = list(inner)
        ahead[d - a] = slice(1, n[a])
        D.append(u[tuple(ahead)] - u[inner])
    D = torch.stack(D)
    if p.regulariser == api.REG_DIFFUSION:
        R = (D * D).sum()
    elif p.regulariser == api.REG_ANISO_TV:
        R = D.abs().sum()
    else:
        R = (D * D).sum(dim=(0, 1)).sqrt().sum()
    L = S + float(np.float32(p.lambda_diff)) * R / math.prod(m - 1 for m in n)
    (g,) = torch.autograd.grad(L, th)
    return L.detach(), g


def exact(case, seed):
    if case["kind"] == "pair":
        p = _problem(case)
        return _exact_pair(p, *_pair_inputs(p, seed))
    if case["kind"] == "batch":
        got = [_exact_pair(p, *_pair_inputs(p, seed * 1009 + i))
               for i, p in enumerate(_batch_problems(case))]
        return torch.stack([v for v, _ in got]), [g for _, g in got]
    cin, cout, g, x, w, b, dy = _conv_inputs(case, seed)
    B = case["batch"]
    x5 = x.double().reshape(B, g, g, g, cin)
    dy5 = dy.double().reshape(B, g, g, g, cout)
    xp = tnf.pad(x5, (0, 0, 1, 1, 1, 1, 1, 1))
    dyp = tnf.pad(dy5, (0, 0, 1, 1, 1, 1, 1, 1))
    wd = w.double()
    y = torch.zeros((B * g ** 3, cout), dtype=torch.float64, device=DEV)
    dx = torch.zeros((B * g ** 3, cin), dtype=torch.float64, device=DEV)
    dw = torch.zeros((cout, 27, cin), dtype=torch.float64, device=DEV)
    dyf = dy5.reshape(-1, cout).t().contiguous()
    for t in range(27):
        z, yy, xx = t // 9, (t // 3) % 3, t % 3
        xs = xp[:, z:z + g, yy:yy + g, xx:xx + g].reshape(-1, cin)
        y += xs @ wd[:, t].t().contiguous()
        dw[:, t] = dyf @ xs
        ds = dyp[:, 2 - z:2 - z + g, 2 - yy:2 - yy + g, 2 - xx:2 - xx + g].reshape(-1, cout)
        dx += ds @ wd[:, t].contiguous()
    y = y + b.double()
    y = torch.where(y > 0, y, 0.1 * y)
    dx = torch.where(x.double() > 0, dx, 0.1 * dx)
    return y, dx, dw.reshape(cout, 27 * cin), dyf.sum(dim=1)
