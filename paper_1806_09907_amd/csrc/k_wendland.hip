// Wendland basis (Sec. III-C, psi_{3,2} with a support radius sigma per axis)
// expanded onto the voxel grid, u = B theta (Sec. II-A eq. kernel_basis), and
// its transpose, B^T g.
//
// Control j sits at (j - m) delta on each axis, so the lattice is aligned
// with voxel cells of size delta: voxel x = c delta + r (cell c, phase r in
// [0, delta)) sees exactly the controls j = c + qq, qq in [0, K), with the
// weight W[qq][r] = psi(||(r - (qq - m) delta) / sigma||), the same for
// every cell. Both directions are therefore per-cell contractions with one
// fixed table, built once per plan on the host:
//   expand:    u(c, r) = sum_qq W[qq][r] theta(c + qq)
//   transpose: H(qq, c) = sum_r W[qq][r] g(c, r) (in two partial sums over
//              halves of the phases);
//              out(j)   = sum_qq H(j - qq, qq)   over cells inside the grid.
// No kernel value is evaluated on the device.
#include "device_common.h"

namespace air {

namespace {

constexpr int kWCells = 16;  // cells along x per wave (one MFMA tile; both contractions)
constexpr int kWaves = kBlock / 64;
constexpr int kTSplit = 2;   // blocks sharing one cell group's phases in the transpose

// theta -> zero-padded copy [d][ncp_z][ncp_y][ncp_x], scaled.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_wend_pad(const PairDesc P, const float* __restrict__ theta, float scale,
           float* __restrict__ thp) {
    const long long nx = P.wncp[0], ny = P.wncp[1], nz = P.wncp[2];
    const long long tot = DIM * nx * ny * nz;
    const long long NC = (long long)P.nc[0] * P.nc[1] * P.nc[2];
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < tot;
         i += (long long)gridDim.x * kBlock) {
        const int jx = (int)(i % nx);
        const int jy = (int)((i / nx) % ny);
        const long long rest = i / (nx * ny);
        const int jz = (int)(rest % nz);
        const int c = (int)(rest / nz);
        float v = 0.f;
        if (jx < P.nc[0] && jy < P.nc[1] && jz < P.nc[2])
            v = scale * theta[c * NC + ((long long)jz * P.nc[1] + jy) * P.nc[0] + jx];
        thp[i] = v;
    }
}

// Per-axis coordinates (x fastest) of a linear index i in an nx x ny x .
// grid, and their update for i += 4 (the step of every lane in the loops
// below), so that no loop divides.
struct Idx3 {
    int x, y, z;
};
__device__ inline Idx3 idx3(int i, int nx, int ny) {
    return Idx3{i % nx, (i / nx) % ny, i / (nx * ny)};
}
__device__ inline void idx3_add(Idx3& c, int step, int nx, int ny) {
    c.x += step;
    while (c.x >= nx) {
        c.x -= nx;
        ++c.y;
    }
    while (c.y >= ny) {
        c.y -= ny;
        ++c.z;
    }
}
__device__ inline void idx3_add4(Idx3& c, int nx, int ny) {
    c.x += 4;
    while (c.x >= nx) {
        c.x -= nx;
        ++c.y;
    }
    while (c.y >= ny) {
        c.y -= ny;
        ++c.z;
    }
}

// Both contractions run on v_mfma_f32_16x16x4f32 (full FP32). Lane l holds
// A[l % 16][l / 16] of the 16x4 A tile, B[l / 16][l % 16] of the 4x16 B tile
// and D[4 (l / 16) + v][l % 16], v = 0..3, of the 16x16 result.
__device__ inline v4f mfma4(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// u(c, r) = sum_qq W[qq][r] thp(c + qq): per wave M = 64 phases (4 tiles),
// N = kWCells cells (one tile per component), K = the controls qq.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_wend_expand(const PairDesc P, const float* __restrict__ W, const float* __restrict__ thp,
              float* __restrict__ u) {
    const int lane = threadIdx.x & 63;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + (threadIdx.x >> 6));
    const int npc = P.wpad[0] / 64;             // phase chunks
    const int ngx = cdiv(P.wncell[0], kWCells);
    const int ngroups = ngx * P.wncell[1] * P.wncell[2];
    if (gw >= ngroups * npc) return;
    const int pc = gw % npc;
    const int g = gw / npc;
    const int cx0 = (g % ngx) * kWCells;
    const int cy = (g / ngx) % P.wncell[1];
    const int cz = g / (ngx * P.wncell[1]);
    const int Ppad = P.wpad[0];
    const int Q = P.wK[0] * P.wK[1] * P.wK[2];
    const long long sx = P.wncp[0], sy = (long long)P.wncp[0] * P.wncp[1];
    const long long NCp = sy * P.wncp[2];
    v4f acc[4][DIM];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < DIM; ++c) acc[m][c] = v4f{0.f, 0.f, 0.f, 0.f};
    const float* Wr = W + pc * 64 + i16;
    const int isy = (int)sy, isx = (int)sx, incp = (int)NCp;   // offsets fit in 32 bits
    const float* thb = thp + cx0 + i16;
    // operands of the K step whose control for this lane is q (coordinates
    // qc). Branch-free: a control past Q reads a valid address and is zeroed
    // where it is used, so the loads stay in flight until then.
    auto load = [&](int q, const Idx3& qc, float* a, float* b, bool& ok) {
        const int qw = min(q, P.wpad[1] - 1);  // rows >= Q are 0; past the end: clamped
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] = Wr[qw * Ppad + m * 16];
        ok = q < Q;
        // a mask, not a branch: the loads must not wait for a join
        const int off = ((cz + qc.z) * isy + (cy + qc.y) * isx + qc.x) & -(int)ok;
#pragma unroll
        for (int c = 0; c < DIM; ++c) b[c] = thb[off + c * incp];
    };
    auto step = [&](const float* a, const float* b, bool ok) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int c = 0; c < DIM; ++c) acc[m][c] = mfma4(a[m], ok ? b[c] : 0.f, acc[m][c]);
    };
    // two operand sets rotate over an even number of K steps (a padding step
    // past Q contributes 0): each set is reloaded right after its MFMAs
    // issue, so its loads have a whole step of MFMAs to land
    const int nst = ((Q + 3) / 4 + 1) & ~1;
    Idx3 qn = idx3(k4, P.wK[0], P.wK[1]);
    float a0[4], b0[DIM], a1[4], b1[DIM];
    bool ok0, ok1;
    load(k4, qn, a0, b0, ok0);
    for (int st = 0; st < nst; st += 2) {
        idx3_add4(qn, P.wK[0], P.wK[1]);
        load((st + 1) * 4 + k4, qn, a1, b1, ok1);
        step(a0, b0, ok0);
        idx3_add4(qn, P.wK[0], P.wK[1]);
        load((st + 2) * 4 + k4, qn, a0, b0, ok0);
        step(a1, b1, ok1);
    }
    const int P3 = P.sp[0] * P.sp[1] * P.sp[2];
    const long long N = P.nvox;
    const int x0 = (cx0 + i16) * P.sp[0];
    // phases r = pc 64 + 16 m + 4 k4 + v in increasing order, coordinates stepped
    Idx3 rc = idx3(pc * 64 + 4 * k4, P.sp[0], P.sp[1]);
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (m + v > 0) idx3_add(rc, v == 0 ? 13 : 1, P.sp[0], P.sp[1]);
            const int r = pc * 64 + m * 16 + 4 * k4 + v;
            if (r >= P3) continue;
            const int x = x0 + rc.x, y = cy * P.sp[1] + rc.y, z = cz * P.sp[2] + rc.z;
            if (x >= P.n[0] || y >= P.n[1] || z >= P.n[2]) continue;
            const long long vox = ((long long)z * P.n[1] + y) * P.n[0] + x;
#pragma unroll
            for (int c = 0; c < DIM; ++c) u[c * N + vox] = acc[m][c][v];
        }
}

// H(qq, c) = sum_r W[qq][r] g(c, r) for kWCells cells along x and 64 values
// of qq: per wave M = 64 qq (4 tiles), N = kWCells cells (one tile per
// component), K = the phases, split over the block's waves; the waves'
// results are added in LDS in a fixed order.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_wend_cells_t(const PairDesc P, const float* __restrict__ WT, const float* __restrict__ g,
               float* __restrict__ H) {
    constexpr int NA = 4 * DIM * 4;   // accumulator floats per lane
    __shared__ float red[kWaves * 64 * NA];
    const int lane = threadIdx.x & 63;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int w = threadIdx.x >> 6;
    const int nqc = P.wpad[1] / 64;
    const int ngx = cdiv(P.wncell[0], kWCells);
    const int part = blockIdx.x % kTSplit;     // which share of the phases
    const int qc = (blockIdx.x / kTSplit) % nqc;
    const int grp = blockIdx.x / (kTSplit * nqc);
    const int cx0 = (grp % ngx) * kWCells;
    const int cy = (grp / ngx) % P.wncell[1];
    const int cz = grp / (ngx * P.wncell[1]);
    const int Qpad = P.wpad[1];
    const int P3 = P.sp[0] * P.sp[1] * P.sp[2];
    const int nstep = P.wpad[0] / 4;
    const int nsub = kTSplit * kWaves;         // K ranges: one per wave of the split blocks
    const int s0 = (part * kWaves + w) * nstep / nsub, s1 = (part * kWaves + w + 1) * nstep / nsub;
    const long long N = P.nvox;
    const int cxl = cx0 + i16;                 // this lane's cell of the B tile
    const bool cell_ok = cxl < P.wncell[0];
    v4f acc[4][DIM];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < DIM; ++c) acc[m][c] = v4f{0.f, 0.f, 0.f, 0.f};
    const float* Wq = WT + qc * 64 + i16;
    const int nx = P.n[0], nxy = P.n[0] * P.n[1], iN = (int)N;  // < 2^31 (plan check)
    const int bx = cxl * P.sp[0], by = cy * P.sp[1], bz = cz * P.sp[2];
    // operands of the K step whose phase for this lane is r (coordinates rc).
    // Branch-free: a phase outside the grid reads voxel 0 and is zeroed where
    // it is used, so the loads stay in flight until then.
    auto load = [&](int r, const Idx3& rc, float* a, float* b, bool& ok) {
        const int rw = min(r, P.wpad[0] - 1);  // rows >= P3 are 0; past the end: clamped
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] = Wq[rw * Qpad + m * 16];
        const int x = bx + rc.x, y = by + rc.y, z = bz + rc.z;
        ok = r < P3 && cell_ok && x < P.n[0] && y < P.n[1] && z < P.n[2];
        // a mask, not a branch: the loads must not wait for a join
        const int vox = (z * nxy + y * nx + x) & -(int)ok;
#pragma unroll
        for (int c = 0; c < DIM; ++c) b[c] = g[c * iN + vox];
    };
    auto step = [&](const float* a, const float* b, bool ok) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int c = 0; c < DIM; ++c) acc[m][c] = mfma4(a[m], ok ? b[c] : 0.f, acc[m][c]);
    };
    // two operand sets rotate over an even number of K steps (a padding step
    // past this wave's range contributes 0): each set is reloaded right after
    // its MFMAs issue, so its loads have a whole step of MFMAs to land
    const int s2 = s0 + ((s1 - s0 + 1) & ~1);
    Idx3 rn = idx3(s0 * 4 + k4, P.sp[0], P.sp[1]);
    float a0[4], b0[DIM], a1[4], b1[DIM];
    bool ok0, ok1;
    load(s0 * 4 + k4, rn, a0, b0, ok0);
    ok0 = ok0 && s0 < s1;
    for (int st = s0; st < s2; st += 2) {
        idx3_add4(rn, P.sp[0], P.sp[1]);
        load((st + 1) * 4 + k4, rn, a1, b1, ok1);
        ok1 = ok1 && st + 1 < s1;
        step(a0, b0, ok0);
        idx3_add4(rn, P.sp[0], P.sp[1]);
        load((st + 2) * 4 + k4, rn, a0, b0, ok0);
        ok0 = ok0 && st + 2 < s1;
        step(a1, b1, ok1);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < DIM; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(w * 64 + lane) * NA + (m * DIM + c) * 4 + v] = acc[m][c][v];
    __syncthreads();
    const int Q = P.wK[0] * P.wK[1] * P.wK[2];
    const long long ncells = (long long)P.wncell[0] * P.wncell[1] * P.wncell[2];
    const long long row = ((long long)cz * P.wncell[1] + cy) * P.wncell[0] + cx0;
    // consecutive threads take consecutive cells of one (component, qq) row
    for (int o = threadIdx.x; o < 64 * kWCells * DIM; o += kBlock) {
        const int t = o % kWCells;
        const int c = (o / kWCells) % DIM;
        const int ql = o / (kWCells * DIM);
        const int m = ql / 16, k4o = (ql % 16) / 4, v = ql % 4;
        const int src = (k4o * 16 + t) * NA + (m * DIM + c) * 4 + v;
        float sum = 0.f;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) sum += red[ww * 64 * NA + src];
        const int qv = qc * 64 + ql;
        if (qv < Q && cx0 + t < P.wncell[0])
            H[(((long long)part * DIM + c) * Q + qv) * ncells + row + t] = sum;
    }
}

// out(j) (+)= scale * sum_qq H(j - qq, qq) over cells inside the grid, with
// H laid out [d][K^d][cells]. A block takes 64 consecutive controls (one per
// lane, so a wave reads consecutive cells) and splits qq over its waves; the
// partial sums are added in a fixed order.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_wend_gather(const PairDesc P, const float* __restrict__ H, float scale, int accumulate,
              float* __restrict__ out) {
    __shared__ float red[kWaves][64];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const long long NC = (long long)P.nc[0] * P.nc[1] * P.nc[2];
    const long long ncells = (long long)P.wncell[0] * P.wncell[1] * P.wncell[2];
    const int Q = P.wK[0] * P.wK[1] * P.wK[2];
    const long long i = (long long)blockIdx.x * 64 + lane;   // (component, control)
    float s = 0.f;
    if (i < DIM * NC) {
        const int c = (int)(i / NC);
        const long long j = i % NC;
        const int jx = (int)(j % P.nc[0]);
        const int jy = (int)((j / P.nc[0]) % P.nc[1]);
        const int jz = (int)(j / ((long long)P.nc[0] * P.nc[1]));
        const long long hpart = (long long)DIM * Q * ncells;   // one share of the phases
        const float* Hc = H + (long long)c * Q * ncells;
        Idx3 qi = idx3(w, P.wK[0], P.wK[1]);
        for (int qq = w; qq < Q; qq += kWaves, idx3_add4(qi, P.wK[0], P.wK[1])) {
            const int cx = jx - qi.x, cy = jy - qi.y, cz = jz - qi.z;
            if (cx < 0 || cx >= P.wncell[0] || cy < 0 || cy >= P.wncell[1] || cz < 0 ||
                cz >= P.wncell[2])
                continue;
            const long long o =
                (long long)qq * ncells + ((long long)cz * P.wncell[1] + cy) * P.wncell[0] + cx;
#pragma unroll
            for (int pt = 0; pt < kTSplit; ++pt) s += Hc[pt * hpart + o];
        }
    }
    red[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < DIM * NC) {
        float t = 0.f;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) t += red[ww][lane];
        const float v = scale * t;
        out[i] = accumulate ? out[i] + v : v;
    }
}

// ---- 3D grids whose cells see 4 controls per axis (cubic B-splines; Wendland
// with sigma up to 2 spacings): the same contractions with every operand of a
// wave's product in flight at once.

// The controls of one 16-cell group are read from theta itself (a control
// past the grid reads past the buffer, which gives zero), 16-byte stores
// write four phases along x at once where the spacing allows it (VEC: a
// multiple of 4). A K step is one (qz, qy) row of controls, its four k the
// qx, in the order of k_wend_expand, so u is the same bit for bit. All 112
// loads of a wave are issued before their products; k_wend_expand waits for
// each step's. 128^3, spacing 8: 24.1 us
// and 4.7 for the padded copy -> 15-16 us (5.1 us of MFMA issue).
template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_cell_expand4(const PairDesc P, const float* __restrict__ W, const float* __restrict__ theta,
               float scale, float* __restrict__ u) {
    const int lane = threadIdx.x & 63;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + (threadIdx.x >> 6));
    const int npc = P.wpad[0] / 64;             // phase chunks
    const int ngx = cdiv(P.wncell[0], kWCells);
    if (gw >= ngx * P.wncell[1] * P.wncell[2] * npc) return;
    const int pc = gw % npc;
    const int g = gw / npc;
    const int cx0 = (g % ngx) * kWCells;
    const int cy = (g / ngx) % P.wncell[1];
    const int cz = g / (ngx * P.wncell[1]);
    const int Ppad = P.wpad[0];
    const long long NC = (long long)P.nc[0] * P.nc[1] * P.nc[2];
    __amdgpu_buffer_rsrc_t rT[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) rT[c] = make_rsrc(theta + c * NC, (uint32_t)(NC * 4));
    const int jx = cx0 + i16 + k4;
    const int vo = jx < P.nc[0] ? jx * 4 : kNoElem;
    const float* Wr = W + k4 * Ppad + pc * 64 + i16;
    float a[16][4], b[16][3];
#pragma unroll
    for (int st = 0; st < 16; ++st) {
        const int jz = cz + (st >> 2), jy = cy + (st & 3);
        const bool in = jz < P.nc[2] && jy < P.nc[1];   // uniform
        const int so = in ? (jz * P.nc[1] + jy) * P.nc[0] * 4 : 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) b[st][c] = load1(rT[c], in ? vo : kNoElem, so);
#pragma unroll
        for (int m = 0; m < 4; ++m) a[st][m] = Wr[st * 4 * Ppad + m * 16];
    }
    v4f acc[4][3];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[m][c] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 16; ++st)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float bc = scale * b[st][c];
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[m][c] = mfma4(a[st][m], bc, acc[m][c]);
        }
    const int P3 = P.sp[0] * P.sp[1] * P.sp[2];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2], iN = (int)P.nvox;
    const int x0 = (cx0 + i16) * P.sp[0], y0 = cy * P.sp[1], z0 = cz * P.sp[2];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int r0 = pc * 64 + m * 16 + 4 * k4;   // this lane's phases r0 .. r0 + 3
        if constexpr (VEC) {
            if (r0 >= P3) continue;
            const Idx3 rc = idx3(r0, P.sp[0], P.sp[1]);
            const int x = x0 + rc.x, y = y0 + rc.y, z = z0 + rc.z;
            if (x >= nx || y >= ny || z >= nz) continue;
            const int vox = (z * ny + y) * nx + x;
            if (x + 3 < nx) {
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    __builtin_memcpy(u + (long long)c * iN + vox, &acc[m][c], 16);
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int v = 0; v < 3; ++v)
                        if (x + v < nx) u[(long long)c * iN + vox + v] = acc[m][c][v];
            }
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (r0 + v >= P3) continue;
                const Idx3 rc = idx3(r0 + v, P.sp[0], P.sp[1]);
                const int x = x0 + rc.x, y = y0 + rc.y, z = z0 + rc.z;
                if (x >= nx || y >= ny || z >= nz) continue;
                const int vox = (z * ny + y) * nx + x;
#pragma unroll
                for (int c = 0; c < 3; ++c) u[(long long)c * iN + vox] = acc[m][c][v];
            }
        }
    }
}

// The transpose. A block of eight waves takes one 16-cell group; wave w the
// phase chunks w, w + 8, .., 64 phases each. A lane loads four phases of its
// cell at once (VEC: one 16-byte load), K step j of 16 phases being phase j
// of every lane's four. The waves' products are added in LDS in a fixed
// order, and H is summed over qx there:
//   Hx(c, qz, qy, cz, cy, group, i) = sum_qx H(cell 16 group + i - qx, q),
// i < 19, stored with pitch kHx, a third of H, so the gather reads 16 to 32
// values per control instead of 128. 128^3, spacing 8: 18.9
// and 10.4 us for the gather -> 14.3 and 4.0.
constexpr int kHx = 20;
constexpr int kCellTBlock = 512;
template <bool VEC>
__global__ void __launch_bounds__(kCellTBlock)
k_cell_t4(const PairDesc P, const float* __restrict__ WT, const float* __restrict__ g,
          float* __restrict__ Hx) {
    constexpr int NW = kCellTBlock / 64, NA = 48;
    __shared__ float red[NW / 2][NA][64];
    const int lane = threadIdx.x & 63;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ngx = cdiv(P.wncell[0], kWCells);
    const int grp = blockIdx.x % ngx, cy = (blockIdx.x / ngx) % P.wncell[1];
    const int cz = blockIdx.x / (ngx * P.wncell[1]);
    const int npc = P.wpad[0] / 64, Qpad = P.wpad[1];
    const int P3 = P.sp[0] * P.sp[1] * P.sp[2];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const long long N = P.nvox;
    const int cxl = grp * kWCells + i16;
    const int x0 = cxl * P.sp[0], y0 = cy * P.sp[1], z0 = cz * P.sp[2];
    __amdgpu_buffer_rsrc_t rg[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) rg[c] = make_rsrc(g + c * N, (uint32_t)(N * 4));
    v4f acc[4][3];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[m][c] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int pc = w; pc < npc; pc += NW) {
        v4f b[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r0 = pc * 64 + 16 * q + 4 * k4;
            if constexpr (VEC) {
                const Idx3 rc = idx3(r0, P.sp[0], P.sp[1]);
                const int x = x0 + rc.x, y = y0 + rc.y, z = z0 + rc.z;
                const bool ok = r0 < P3 && x < nx && y < ny && z < nz;
                const int vo = ok ? ((z * ny + y) * nx + x) * 4 : kNoElem;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    v4f v = __builtin_bit_cast(
                        v4f, __builtin_amdgcn_raw_buffer_load_b128(rg[c], vo, 0, 0));
                    // past the row's end: the next row's voxels
#pragma unroll
                    for (int e = 1; e < 4; ++e) v[e] = x + e < nx ? v[e] : 0.f;
                    b[q][c] = v;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const Idx3 rc = idx3(r0 + e, P.sp[0], P.sp[1]);
                    const int x = x0 + rc.x, y = y0 + rc.y, z = z0 + rc.z;
                    const bool ok = r0 + e < P3 && x < nx && y < ny && z < nz;
                    const int vo = ok ? ((z * ny + y) * nx + x) * 4 : kNoElem;
#pragma unroll
                    for (int c = 0; c < 3; ++c) b[q][c][e] = load1(rg[c], vo, 0);
                }
            }
        }
        float a[16][4];
        const float* Wq = WT + (pc * 64 + 4 * k4) * Qpad + i16;   // rows >= P3 are zero
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < 4; ++m) a[4 * q + e][m] = Wq[(16 * q + e) * Qpad + 16 * m];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        acc[m][c] = mfma4(a[4 * q + e][m], b[q][c][e], acc[m][c]);
    }
    if (w >= NW / 2) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[w - NW / 2][(m * 3 + c) * 4 + v][lane] = acc[m][c][v];
    }
    __syncthreads();
    if (w < NW / 2) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[w][(m * 3 + c) * 4 + v][lane] += acc[m][c][v];
    }
    __syncthreads();
    // control q = 4 (4 m + k4) + v of the products is (qz, qy) = (m, k4), qx = v
    for (int o = threadIdx.x; o < 16 * 3 * kHx; o += kCellTBlock) {
        const int i = o % kHx, rest = o / kHx;
        const int c = rest % 3, qyz = rest / 3;
        float s = 0.f;
#pragma unroll
        for (int qx = 0; qx < 4; ++qx) {
            const int t = i - qx;
            if (t < 0 || t >= kWCells) continue;
#pragma unroll
            for (int ww = 0; ww < NW / 2; ++ww)
                s += red[ww][((qyz >> 2) * 3 + c) * 4 + qx][(qyz & 3) * 16 + t];
        }
        Hx[((((long long)c * 16 + qyz) * P.wncell[2] + cz) * P.wncell[1] + cy) * ngx * kHx +
           grp * kHx + i] = s;
    }
}

// out(j) (+)= scale * the sum of Hx over the (qz, qy) and groups that hold
// control j. As in k_wend_gather, 64 controls per block, (qz, qy) split over
// the waves.
__global__ void __launch_bounds__(kBlock)
k_cell_gather4(const PairDesc P, const float* __restrict__ Hx, float scale, int accumulate,
               float* __restrict__ out) {
    __shared__ float red[kWaves][64];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int NC = P.nc[0] * P.nc[1] * P.nc[2];
    const int ngx = cdiv(P.wncell[0], kWCells);
    const long long i = (long long)blockIdx.x * 64 + lane;   // (component, control)
    float s = 0.f;
    if (i < 3LL * NC) {
        const int c = (int)(i / NC), j = (int)(i - (long long)c * NC);
        const int jx = j % P.nc[0], jyz = j / P.nc[0];
        const int jy = jyz % P.nc[1], jz = jyz / P.nc[1];
        const int ghi = min(jx / kWCells, ngx - 1), glo = jx > 18 ? (jx - 3) / kWCells : 0;
#pragma unroll
        for (int k = 0; k < 16 / kWaves; ++k) {
            const int qyz = w * (16 / kWaves) + k;
            const int cz = jz - (qyz >> 2), cy = jy - (qyz & 3);
            if (cz < 0 || cz >= P.wncell[2] || cy < 0 || cy >= P.wncell[1]) continue;
            const float* h = Hx + ((((long long)c * 16 + qyz) * P.wncell[2] + cz) * P.wncell[1] +
                                   cy) * ngx * kHx;
            for (int gi = glo; gi <= ghi; ++gi)
                if (jx - gi * kWCells < kWCells + 3) s += h[gi * kHx + jx - gi * kWCells];
        }
    }
    red[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < 3LL * NC) {
        float t = 0.f;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) t += red[ww][lane];
        const float v = scale * t;
        out[i] = accumulate ? out[i] + v : v;
    }
}

// Whether the kernels above can take the plan: 3D, four controls per axis,
// byte offsets in 32 bits, and at least three cells along x (with fewer, Hx
// would not fit in the workspace of H).
__host__ inline bool cells4(const PairDesc& P, int dim) {
    return dim == 3 && P.wK[0] == 4 && P.wK[1] == 4 && P.wK[2] == 4 && P.wncell[0] >= 3 &&
           (long long)P.nc[0] * P.nc[1] * P.nc[2] <= kMaxVoxels;
}

// Where they are the faster ones (general kernels, these; us with the padded
// copy and the gather). Phases along x that are no multiple of 4 are loaded
// and stored one by one, which only pays while the launch does not fill the
// chip's queues: up to kCells4Voxels (spacing 10 at 128^3 29 and 15, at 200^3
// 97 and 103). The transpose gives a 16-cell group to one block, so coarse
// grids of few groups leave the chip idle longer than the general kernel's two
// blocks (spacing 16 at 64^3 67 and 71, 32 at 128^3 408 and 510, but 12 at 64^3
// 37 and 36): up to 12^3 phases, or at least 128 groups (16 at 180^3 97 and
// 77); up to 10^3 where phases go one by one (10 at 64^3 28 and 27, 13 at 64^3
// 44 and 51).
constexpr long long kCells4Voxels = 1LL << 22;
__host__ inline bool cells4_expand_pays(const PairDesc& P) {
    return P.sp[0] % 4 == 0 || P.nvox <= kCells4Voxels;
}
__host__ inline bool cells4_transpose_pays(const PairDesc& P) {
    const int phases = P.sp[0] * P.sp[1] * P.sp[2];
    if (P.sp[0] % 4) return phases <= 1000 && P.nvox <= kCells4Voxels;
    const long long groups =
        (long long)cdiv(P.wncell[0], kWCells) * P.wncell[1] * P.wncell[2];
    return phases <= 1728 || groups >= 128;
}

__host__ inline int wend_grid(long long n) {
    const long long b = (n + kBlock - 1) / kBlock;
    return (int)(b < 4096 ? (b < 1 ? 1 : b) : 4096);
}

}  // namespace

// u = scale * B theta. thp: d * prod(wncp) floats of workspace; W: the
// [wpad0][...] table in the plan's constants.
hipError_t launch_wendland_expand(const PairDesc& P, const float* consts_dev, int dim,
                                  const float* theta, float scale, float* thp, float* u,
                                  hipStream_t s) {
    const long long np = (long long)dim * P.wncp[0] * P.wncp[1] * P.wncp[2];
    const float* W = consts_dev + P.wend_off[0];
    const int ngx = cdiv(P.wncell[0], kWCells);
    const long long waves = (long long)ngx * P.wncell[1] * P.wncell[2] * (P.wpad[0] / 64);
    const int blocks = (int)((waves + kWaves - 1) / kWaves);
    if (cells4(P, dim) && cells4_expand_pays(P)) {
        if (P.sp[0] % 4 == 0)
            hipLaunchKernelGGL(k_cell_expand4<true>, dim3(blocks), dim3(kBlock), 0, s, P, W,
                               theta, scale, u);
        else
            hipLaunchKernelGGL(k_cell_expand4<false>, dim3(blocks), dim3(kBlock), 0, s, P, W,
                               theta, scale, u);
    } else if (dim == 3) {
        hipLaunchKernelGGL(k_wend_pad<3>, dim3(wend_grid(np)), dim3(kBlock), 0, s, P, theta,
                           scale, thp);
        hipLaunchKernelGGL(k_wend_expand<3>, dim3(blocks), dim3(kBlock), 0, s, P, W, thp, u);
    } else {
        hipLaunchKernelGGL(k_wend_pad<2>, dim3(wend_grid(np)), dim3(kBlock), 0, s, P, theta,
                           scale, thp);
        hipLaunchKernelGGL(k_wend_expand<2>, dim3(blocks), dim3(kBlock), 0, s, P, W, thp, u);
    }
    return hipGetLastError();
}

// grad (+)= scale * B^T g. H: wendland_h_parts() * d * K^d * prod(wncell)
// floats of workspace.
hipError_t launch_wendland_adjoint(const PairDesc& P, const float* consts_dev, int dim,
                                   const float* g, float scale, float* H, float* grad,
                                   bool accumulate, hipStream_t s) {
    const float* WT = consts_dev + P.wend_off[1];
    const int ngx = cdiv(P.wncell[0], kWCells);
    const int blocks = ngx * P.wncell[1] * P.wncell[2] * (P.wpad[1] / 64) * kTSplit;
    const long long NC = (long long)dim * P.nc[0] * P.nc[1] * P.nc[2];
    const int gblocks = (int)((NC + 63) / 64);
    if (cells4(P, dim) && cells4_transpose_pays(P)) {
        const int groups = ngx * P.wncell[1] * P.wncell[2];
        if (P.sp[0] % 4 == 0)
            hipLaunchKernelGGL(k_cell_t4<true>, dim3(groups), dim3(kCellTBlock), 0, s, P, WT, g, H);
        else
            hipLaunchKernelGGL(k_cell_t4<false>, dim3(groups), dim3(kCellTBlock), 0, s, P, WT, g, H);
        hipLaunchKernelGGL(k_cell_gather4, dim3(gblocks), dim3(kBlock), 0, s, P, H, scale,
                           accumulate ? 1 : 0, grad);
    } else if (dim == 3) {
        hipLaunchKernelGGL(k_wend_cells_t<3>, dim3(blocks), dim3(kBlock), 0, s, P, WT, g, H);
        hipLaunchKernelGGL(k_wend_gather<3>, dim3(gblocks), dim3(kBlock), 0, s, P, H, scale,
                           accumulate ? 1 : 0, grad);
    } else {
        hipLaunchKernelGGL(k_wend_cells_t<2>, dim3(blocks), dim3(kBlock), 0, s, P, WT, g, H);
        hipLaunchKernelGGL(k_wend_gather<2>, dim3(gblocks), dim3(kBlock), 0, s, P, H, scale,
                           accumulate ? 1 : 0, grad);
    }
    return hipGetLastError();
}

// Cells along x per wave in both contractions (the padded control grid is
// rounded up to a multiple of it along x).
int wendland_cells_per_wave() { return kWCells; }
// Partial per-cell sums the transpose writes (summed by the gather).
int wendland_h_parts() { return kTSplit; }

}  // namespace air
