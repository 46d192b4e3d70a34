// LCC (Sec. III-B): the local version of NCC on a dense displacement u.
// For every voxel x of the masked set X' (sample point inside the moving
// image), over the window N(x) = {y in X' : |y - x|_inf <= r}:
//   n, the means muF, muW, the variances varF, varW and the covariance
//   (divided by n), rho(x) = cov / sqrt(varF varW + eps),
//   S = -(1/|X'|) sum_{x in X'} rho(x).
// The statistics come from box sums of m, mF, mW, mF^2, mW^2, mFW (m the
// mask), in FP64 so that E[X^2] - mu^2 does not cancel. Writing
// B = sum mW, D = sum mW^2, E = sum mFW over N(x), V = varF varW + eps:
//   drho/dB = -muF / (n sqrt V) + rho varF muW / (n V)
//   drho/dD = -rho varF / (2 n V)
//   drho/dE = 1 / (n sqrt V)
// and, as y is in N(x) exactly when x is in the window of y,
//   dS/dW(y) = -(1/|X'|) m(y) (box(aB) + 2 W(y) box(aD) + F(y) box(aE))(y)
// with a* = drho/d* on X' and 0 elsewhere. Every box sum is separable: an
// LDS-tiled pass over x and y, then a running sum along z — fused into one
// kernel per direction in 3D for radii up to 4 (the z window as a register
// ring), else as separate passes through FP64 maps.
#include <utility>

#include "device_common.h"

namespace air {

namespace {

constexpr int kTX = 32, kTY = 8;   // xy tile of the box passes (kBlock threads)
constexpr int kZSeg = 16;          // voxels of z walked per thread in the z passes
constexpr double kLccEps = 1e-10;  // eps of the denominator (image units^4)

// Statistics -> rho and the coefficient maps (aB, aD, aE) on X' (two FP64
// divisions per voxel: 1/n and 1/sqrt(V)).
__device__ inline void lcc_coef(const double* s, float* aB, float* aD, float* aE, double* rho) {
    const double in = 1.0 / s[0];
    const double mf = s[1] * in, mw = s[2] * in;
    const double vf = s[3] * in - mf * mf, vw = s[4] * in - mw * mw;
    const double cv = s[5] * in - mf * mw;
    const double V = vf * vw + kLccEps;
    const double isq = 1.0 / sqrt(V);
    const double r = cv * isq;
    const double iV = isq * isq;
    *aB = (float)(in * (r * vf * mw * iV - mf * isq));
    *aD = (float)(-0.5 * r * vf * in * iV);
    *aE = (float)(in * isq);
    *rho = r;
}

// Gathers of one zero-padded sample: the x pairs of its 2^(DIM-1) rows, each
// in one load at the clamped pair start. A row outside the volume reads zeros
// (kNoElem); lo and hi tell which of a pair is the cell's left and right
// element (0 left of the pair, 1 and 2 its elements, 3 right of it).
template <int DIM>
struct Gather {
    float f[3];
    v2f p[1 << (DIM - 1)];
    int lo, hi;
    bool in;
};
template <int DIM>
__device__ inline void gather_issue(const PairDesc& P, __amdgpu_buffer_rsrc_t rM, const int* x,
                                    const float* u, Gather<DIM>& G) {
    int j[3] = {0, 0, 0};
    G.in = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const AxisCell c = axis_cell(x[a], disp_of(u[a], P.s[a]), P.n[a]);
        G.in = G.in & c.in;
        j[a] = c.t;
        G.f[a] = c.f;
    }
    const int tb = min(max(j[0], 0), P.n[0] - 2);
    G.lo = j[0] - tb + 1;
    G.hi = G.lo + 1;
    const bool any = j[0] >= -1 && j[0] < P.n[0];
#pragma unroll
    for (int r = 0; r < (1 << (DIM - 1)); ++r) {
        const int y = j[1] + (r & 1), z = DIM == 3 ? j[2] + (r >> 1) : 0;
        const bool ok = any & (y >= 0) & (y < P.n[1]) & (z >= 0) & (DIM == 2 || z < P.n[2]);
        const int off = ok ? 4 * (tb + P.n[0] * (y + P.n[1] * z)) : kNoElem;
        AIR_CHECK(off == kNoElem || (off >= 0 && off / 4 + 1 < P.nvox), kDbgSampler);
        G.p[r] = load2(rM, off, 0);
    }
}
// The sample and its derivative on the cell (the terms and order of
// sample_general).
template <int DIM>
__device__ inline float gather_value(const Gather<DIM>& G, float* d) {
    float W = 0.f;
#pragma unroll
    for (int a = 0; a < DIM; ++a) d[a] = 0.f;
#pragma unroll
    for (int c = 0; c < (1 << DIM); ++c) {
        const v2f p = G.p[c >> 1];
        const int k = (c & 1) ? G.hi : G.lo;
        const float val = k == 1 ? p.x : k == 2 ? p.y : 0.f;
        float w = 1.f;
#pragma unroll
        for (int a = 0; a < DIM; ++a) w *= ((c >> a) & 1) ? G.f[a] : 1.f - G.f[a];
        W += w * val;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            float wa = ((c >> a) & 1) ? 1.f : -1.f;
#pragma unroll
            for (int b = 0; b < DIM; ++b)
                if (b != a) wa *= ((c >> b) & 1) ? G.f[b] : 1.f - G.f[b];
            d[a] += wa * val;
        }
    }
    return W;
}

// W, the mask and dW/dp (voxel units) at every voxel. Bound by the gathers,
// which cost the same whatever their width: x pairs halve them. A thread
// walks kSampleZ planes of one column (one division, two planes of gathers
// in flight), neighbouring blocks on one XCD. 128^3: eight guarded loads and
// four 64-bit divisions per voxel 20.0 us, this 14.0 us.
constexpr int kSampleZ = 8;
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_lcc_sample(const PairDesc P, const float* __restrict__ M, const float* __restrict__ u,
             float* __restrict__ W, uint8_t* __restrict__ mk, float* __restrict__ dW) {
    constexpr int NB = DIM == 3 ? 2 : 1;   // planes in flight
    const int sz = P.n[0] * P.n[1], ncb = cdiv(sz, kBlock);
    const int item = xcd_item(blockIdx.x, ncb * cdiv(P.n[2], kSampleZ), 0);
    if (item < 0) return;
    const int z0 = item / ncb * kSampleZ, z1 = min(P.n[2], z0 + kSampleZ);
    const int c = (item % ncb) * kBlock + threadIdx.x;
    const bool col = c < sz;
    const int y = c / P.n[0], x = c - y * P.n[0];
    const long long N = P.nvox;
    const uint32_t nb = 4u * (uint32_t)N;
    const __amdgpu_buffer_rsrc_t rM = make_rsrc(M, nb), rW = make_rsrc(W, nb),
                                 rm = make_rsrc(mk, (uint32_t)N);
    __amdgpu_buffer_rsrc_t ru[DIM], rd[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        ru[a] = make_rsrc(u + a * N, nb);
        rd[a] = make_rsrc(dW + a * N, nb);
    }
    for (int zb = z0; zb < z1; zb += NB) {
        Gather<DIM> G[NB];
        float q[NB][DIM];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int vo = col && zb + k < z1 ? 4 * (c + (zb + k) * sz) : kNoElem;
#pragma unroll
            for (int a = 0; a < DIM; ++a) q[k][a] = load1(ru[a], vo, 0);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int xv[3] = {x, y, zb + k};
            gather_issue<DIM>(P, rM, xv, q[k], G[k]);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const bool on = col && zb + k < z1;
            const int v = c + (zb + k) * sz, vo = on ? 4 * v : kNoElem;
            float d[DIM];
            store1(rW, gather_value<DIM>(G[k], d), vo, 0);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(G[k].in ? 1 : 0), rm, on ? v : kNoElem, 0,
                                                 0);
#pragma unroll
            for (int a = 0; a < DIM; ++a) store1(rd[a], d[a], vo, 0);
        }
    }
}

// Box sums over x and y (radius r) of NCH channels at one plane:
// MODE 0: the six statistics channels of (F, W, m); MODE 1: three FP32 maps.
// out: [NCH][N] FP64. Dynamic LDS: the raw tile with halo, then the x sums.
template <int NCH, int MODE>
__global__ void __launch_bounds__(kBlock)
k_lcc_box_xy(const PairDesc P, int r, const float* __restrict__ a0, const float* __restrict__ a1,
             const float* __restrict__ a2, const uint8_t* __restrict__ mk,
             double* __restrict__ out) {
    extern __shared__ double lds[];
    constexpr int NIN = 3;
    const int HX = kTX + 2 * r, HY = kTY + 2 * r;
    float* raw = reinterpret_cast<float*>(lds);            // [NIN][HY][HX]
    double* xs = lds + (NIN * HY * HX + 1) / 2;             // [NCH][HY][kTX]
    const int ntx = cdiv(P.n[0], kTX), nty = cdiv(P.n[1], kTY);
    const int bx = blockIdx.x % ntx, by = (blockIdx.x / ntx) % nty;
    const int z = blockIdx.x / (ntx * nty);
    const int x0 = bx * kTX - r, y0 = by * kTY - r;
    const long long plane = (long long)z * P.n[0] * P.n[1];
    for (int i = threadIdx.x; i < HY * HX; i += kBlock) {
        const int yy = y0 + i / HX, xx = x0 + i % HX;
        float v0 = 0.f, v1 = 0.f, v2 = 0.f;
        if (xx >= 0 && xx < P.n[0] && yy >= 0 && yy < P.n[1]) {
            const long long v = plane + (long long)yy * P.n[0] + xx;
            if (MODE == 0) {
                if (mk[v]) {
                    v0 = 1.f;
                    v1 = a0[v];
                    v2 = a1[v];
                }
            } else {
                v0 = a0[v];
                v1 = a1[v];
                v2 = a2[v];
            }
        }
        raw[i] = v0;
        raw[HY * HX + i] = v1;
        raw[2 * HY * HX + i] = v2;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HY * kTX; i += kBlock) {
        const int ry = i / kTX, tx = i % kTX;
        double s[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) s[c] = 0.0;
        for (int dx = 0; dx <= 2 * r; ++dx) {
            const int k = ry * HX + tx + dx;
            const double e0 = raw[k], e1 = raw[HY * HX + k], e2 = raw[2 * HY * HX + k];
            if (MODE == 0) {
                // m, mF, mW, mF^2, mW^2, mFW (F and W are zero where m is)
                s[0] += e0;
                s[1] += e1;
                s[2] += e2;
                s[3] += e1 * e1;
                s[4 % NCH] += e2 * e2;
                s[5 % NCH] += e1 * e2;
            } else {
                s[0] += e0;
                s[1] += e1;
                s[2] += e2;
            }
        }
#pragma unroll
        for (int c = 0; c < NCH; ++c) xs[(c * HY + ry) * kTX + tx] = s[c];
    }
    __syncthreads();
    const int tx = threadIdx.x % kTX, ty = threadIdx.x / kTX;
    const int x = bx * kTX + tx, y = by * kTY + ty;
    if (x >= P.n[0] || y >= P.n[1]) return;
    const long long v = plane + (long long)y * P.n[0] + x;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        double t = 0.0;
        for (int dy = 0; dy <= 2 * r; ++dy) t += xs[(c * HY + ty + dy) * kTX + tx];
        out[c * P.nvox + v] = t;
    }
}

// Running box sum along z (radius rz) of NCH FP64 channels for one column and
// a segment of kZSeg planes; calls fin(z, v, sums) at every voxel.
template <int NCH, typename Fin>
__device__ inline void z_walk(const PairDesc& P, int rz, const double* __restrict__ S, long long col,
                              int z0, int z1, Fin fin) {
    const long long sz = (long long)P.n[0] * P.n[1];
    const long long N = P.nvox;
    double s[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) s[c] = 0.0;
    for (int zz = max(0, z0 - rz); zz <= min(P.n[2] - 1, z0 + rz); ++zz)
#pragma unroll
        for (int c = 0; c < NCH; ++c) s[c] += S[c * N + zz * sz + col];
    for (int z = z0; z < z1; ++z) {
        fin(z, z * sz + col, s);
        const int za = z + rz + 1, zr = z - rz;
        if (za < P.n[2])
#pragma unroll
            for (int c = 0; c < NCH; ++c) s[c] += S[c * N + za * sz + col];
        if (zr >= 0)
#pragma unroll
            for (int c = 0; c < NCH; ++c) s[c] -= S[c * N + zr * sz + col];
    }
}

// Statistics -> rho and the coefficient maps (aB, aD, aE) on X'; per-block
// partial sums of (count, sum rho) in block order.
__global__ void __launch_bounds__(kBlock)
k_lcc_stats_z(const PairDesc P, int rz, const double* __restrict__ S,
              const float* __restrict__ F, const float* __restrict__ W,
              const uint8_t* __restrict__ mk, float* __restrict__ A, double* __restrict__ part) {
    __shared__ double red[2 * (kBlock / 64)];
    const long long N = P.nvox;
    const long long ncol = (long long)P.n[0] * P.n[1];
    const int nseg = cdiv(P.n[2], kZSeg);
    const long long item = (long long)blockIdx.x * kBlock + threadIdx.x;
    double acc[2] = {0.0, 0.0};
    if (item < ncol * nseg) {
        const long long col = item % ncol;
        const int seg = (int)(item / ncol);
        const int z0 = seg * kZSeg, z1 = min(P.n[2], z0 + kZSeg);
        z_walk<6>(P, rz, S, col, z0, z1, [&](int, long long v, const double* s) {
            float aB = 0.f, aD = 0.f, aE = 0.f;
            if (mk[v]) {
                double rho;
                lcc_coef(s, &aB, &aD, &aE, &rho);
                acc[0] += 1.0;
                acc[1] += rho;
            }
            A[v] = aB;
            A[N + v] = aD;
            A[2 * N + v] = aE;
        });
    }
    block_sum<kBlock, 2>(acc, red);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = acc[0];
        part[2 * blockIdx.x + 1] = acc[1];
    }
}

// value = S (+ lambda * value when lam_acc); scal[0] = 1 / |X'| (0 if empty);
// flags of the pair on an empty mask or a non-finite value.
__global__ void __launch_bounds__(kBlock)
k_lcc_value(const double* __restrict__ part, int nblk, float lambda, int lam_acc, float* value,
            double* scal, uint32_t* flag) {
    __shared__ double red[2 * (kBlock / 64)];
    double s[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < nblk; b += kBlock) {
        s[0] += part[2 * b];
        s[1] += part[2 * b + 1];
    }
    block_sum<kBlock, 2>(s, red);
    if (threadIdx.x == 0) {
        const double cnt = s[0];
        const double S = cnt >= 1.0 ? -s[1] / cnt : 0.0;
        const float v = lam_acc ? (float)(S + (double)lambda * (double)*value) : (float)S;
        *value = v;
        scal[0] = cnt >= 1.0 ? 1.0 / cnt : 0.0;
        uint32_t f = 0;
        if (cnt < 1.0) f |= AIR_FLAG_DEGENERATE;
        if (!isfinite(v)) f |= AIR_FLAG_NONFINITE;
        *flag = f;
    }
}

// g_a = dS/dW dW/dp_a (n_a - 1)/2 on X' (+ lambda g_a when lam_acc).
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_lcc_grad_z(const PairDesc P, int rz, const double* __restrict__ T,
             const float* __restrict__ F, const float* __restrict__ W,
             const uint8_t* __restrict__ mk, const float* __restrict__ dW,
             const double* __restrict__ scal, float lambda, int lam_acc, float* __restrict__ g) {
    const long long N = P.nvox;
    const long long ncol = (long long)P.n[0] * P.n[1];
    const int nseg = cdiv(P.n[2], kZSeg);
    const long long item = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (item >= ncol * nseg) return;
    const long long col = item % ncol;
    const int seg = (int)(item / ncol);
    const int z0 = seg * kZSeg, z1 = min(P.n[2], z0 + kZSeg);
    const double inv = scal[0];
    z_walk<3>(P, rz, T, col, z0, z1, [&](int, long long v, const double* s) {
        float dsdw = 0.f;
        if (mk[v]) dsdw = (float)(-inv * (s[0] + 2.0 * (double)W[v] * s[1] + (double)F[v] * s[2]));
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const float img = dsdw * dW[a * N + v] * P.s[a];
            g[a * N + v] = lam_acc ? fmaf(lambda, g[a * N + v], img) : img;
        }
    });
}

// ---- fused box passes: xy sums in LDS, z window as a register ring ------
// A block owns a kTX x kTY column tile and a chunk of zc output planes. It
// walks the planes of the chunk plus the R-plane halo on each side; for each
// plane it forms the xy box sums of its columns in LDS (as k_lcc_box_xy),
// adds them to a running z sum and subtracts the plane that leaves the
// window, kept in a ring of 2R + 1 slots. The plane loop is unrolled by
// 2R + 1 so that every ring slot is a fixed register.
constexpr int kMaxFusedR = 4;   // radii the register ring covers (3D)

template <int R>
struct Halo {
    static constexpr int HX = kTX + 2 * R, HY = kTY + 2 * R, NI = HX * HY;
    static constexpr int NF = (NI + kBlock - 1) / kBlock;   // tile elements per thread
};

// One plane: both buffers of it (LDS) are used in turn, one barrier a plane.
template <int R, int NCH>
struct XYPlane {
    alignas(16) float raw[3][Halo<R>::NI];   // NI is even: every row starts 8-byte aligned
    alignas(16) double xs[NCH][Halo<R>::HY][kTX];
};

// One plane's tile with halo, as loaded.
template <int R>
struct TileRegs {
    float a[3][Halo<R>::NF];
    uint8_t m[Halo<R>::NF];
};

// The loads of one plane. off: the thread's byte offsets within a plane, the
// same for every plane, kNoElem where the element is outside it; a plane
// outside the volume reads through empty resources. Both give zeros, so the
// loads have no branch and no address arithmetic.
// MODE 0: a0 = F, a1 = W and mk the mask; MODE 1: three FP32 maps.
template <int R, int MODE>
__device__ inline void fetch_tile(const PairDesc& P, const int (&off)[Halo<R>::NF], int zz,
                                  const float* __restrict__ a0, const float* __restrict__ a1,
                                  const float* __restrict__ a2, const uint8_t* __restrict__ mk,
                                  TileRegs<R>& t) {
    using H = Halo<R>;
    const bool zin = zz >= 0 && zz < P.n[2];
    const uint32_t nv = zin ? (uint32_t)P.nvox : 0u;
    const int sv = zin ? zz * P.n[0] * P.n[1] : 0;
    const __amdgpu_buffer_rsrc_t r0 = make_rsrc(a0, 4 * nv), r1 = make_rsrc(a1, 4 * nv);
    const __amdgpu_buffer_rsrc_t r2 = MODE == 0 ? make_rsrc(mk, nv) : make_rsrc(a2, 4 * nv);
#pragma unroll
    for (int it = 0; it < H::NF; ++it) {
        t.a[0][it] = load1(r0, off[it], 4 * sv);
        t.a[1][it] = load1(r1, off[it], 4 * sv);
        if (MODE == 0)
            t.m[it] = load1u8(r2, off[it] == kNoElem ? kNoElem : off[it] >> 2, sv);
        else
            t.a[2][it] = load1(r2, off[it], 4 * sv);
    }
}

// The tile's channels into LDS: MODE 0 (m, mF, mW), MODE 1 the maps, zero
// outside the volume.
template <int R, int NCH, int MODE>
__device__ inline void commit_tile(XYPlane<R, NCH>& L, const TileRegs<R>& t) {
    using H = Halo<R>;
#pragma unroll
    for (int it = 0; it < H::NF; ++it) {
        const int i = threadIdx.x + it * kBlock;
        float v0 = t.a[0][it], v1 = t.a[1][it], v2 = t.a[2][it];
        if (MODE == 0) {
            const bool m = t.m[it] != 0;
            v2 = m ? v1 : 0.f;
            v1 = m ? v0 : 0.f;
            v0 = m ? 1.f : 0.f;
        }
        if (H::NI % kBlock == 0 || i < H::NI) {
            L.raw[0][i] = v0;
            L.raw[1][i] = v1;
            L.raw[2][i] = v2;
        }
    }
}

// x sums of a committed tile. MODE 0 forms m, mF, mW, mF^2, mW^2, mFW (F and
// W are zero where m is). A thread forms two neighbouring x sums, which
// share 2R of their 2R + 1 terms.
template <int R, int NCH, int MODE>
__device__ inline void x_sums(XYPlane<R, NCH>& L) {
    using H = Halo<R>;
    constexpr int XP = kTX / 2;   // pairs of x outputs per row
    constexpr int NE = 2 * R + 2; // raw elements a pair reads
    for (int i = threadIdx.x; i < H::HY * XP; i += kBlock) {
        const int ry = i / XP, tx = 2 * (i % XP);
        float e[3][NE];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < NE; k += 2) {
                const float2 q = *reinterpret_cast<const float2*>(&L.raw[c][ry * H::HX + tx + k]);
                e[c][k] = q.x;
                e[c][k + 1] = q.y;
            }
        double mid[NCH];   // the 2R shared terms
#pragma unroll
        for (int c = 0; c < NCH; ++c) mid[c] = 0.0;
#pragma unroll
        for (int k = 1; k <= 2 * R; ++k) {
            const double e0 = e[0][k], e1 = e[1][k], e2 = e[2][k];
            mid[0] += e0;
            mid[1] += e1;
            mid[2] += e2;
            if (MODE == 0) {
                mid[3 % NCH] = fma(e1, e1, mid[3 % NCH]);
                mid[4 % NCH] = fma(e2, e2, mid[4 % NCH]);
                mid[5 % NCH] = fma(e1, e2, mid[5 % NCH]);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = h ? NE - 1 : 0;
            const double e0 = e[0][k], e1 = e[1][k], e2 = e[2][k];
            double o[NCH];
            o[0] = mid[0] + e0;
            o[1] = mid[1] + e1;
            o[2] = mid[2] + e2;
            if (MODE == 0) {
                o[3 % NCH] = fma(e1, e1, mid[3 % NCH]);
                o[4 % NCH] = fma(e2, e2, mid[4 % NCH]);
                o[5 % NCH] = fma(e1, e2, mid[5 % NCH]);
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c) L.xs[c][ry][tx + h] = o[c];
        }
    }
}

// The y sums of the x sums. Three channels: the thread's own column, row
// threadIdx.x / kTX. Six: the halves of a wave hold its two rows (kTX = 32),
// and there each half sums three of the channels for both rows, which share
// 2R of their 2R + 1 terms (24 reads and adds of LDS instead of 42 at R =
// 3); out = [row of the wave][channel of the half], own_row() gives each
// thread all six channels of its row again.
template <int R, int NCH>
__device__ inline void y_sums(const XYPlane<R, NCH>& L, double* out) {
    const int tx = threadIdx.x % kTX, ty = threadIdx.x / kTX;
    if constexpr (NCH == 6) {
        const int h = ty & 1, y0 = ty & ~1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double* xs = &L.xs[3 * h + c][y0][tx];
            double t = 0.0;
#pragma unroll
            for (int dy = 1; dy <= 2 * R; ++dy) t += xs[dy * kTX];
            out[c] = t + xs[0];
            out[3 + c] = t + xs[(2 * R + 1) * kTX];
        }
    } else {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            double t = 0.0;
#pragma unroll
            for (int dy = 0; dy <= 2 * R; ++dy) t += L.xs[c][ty + dy][tx];
            out[c] = t;
        }
    }
}
template <int NCH>
__device__ inline void own_row(const double* z, double* s) {
    if constexpr (NCH == 6) {
        // the upper half's first row changes places with the lower half's second
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint64_t a = __builtin_bit_cast(uint64_t, z[c]);
            const uint64_t b = __builtin_bit_cast(uint64_t, z[3 + c]);
            const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32),
                                                             false, false);
            s[c] = __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32));
            s[3 + c] = __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
        }
    } else {
#pragma unroll
        for (int c = 0; c < NCH; ++c) s[c] = z[c];
    }
}

template <typename F, int... K>
__device__ inline void for_slots(const F& f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K>()), ...);
}

// Walk the planes of a chunk [z0, z1). fin(z, sums) ends output plane z;
// pre(z) issues the loads of z's per-voxel inputs one plane before. Plane p
// is fetched two planes ahead of its y sums and committed one ahead: its x
// sums run beside the y sums of p - 1, with one barrier between. raw[p & 1]
// is rewritten by p + 2 after the barrier of p, xs[p & 1] after that of
// p + 1, so every reader has passed. No load or store is under a branch: the
// waits stay exact counts, not one for everything in flight.
// With per-element bounds branches, 64-bit addresses, two barriers a plane,
// blocks dealt over the XCDs and every load and store waited for together,
// 128^3 at r = 3 took 48.9 us (statistics) and 48.0 us (gradient); now 42.8
// and 32.3 us. The statistics are bound by FP64 adds and LDS reads together
// (about half the cycles each, two waves a SIMD).
template <int R, int NCH, int MODE, typename Pre, typename Fin>
__device__ inline void z_ring_walk(const PairDesc& P, XYPlane<R, NCH>* L, int bx, int by, int z0,
                                   int z1, const float* a0, const float* a1, const float* a2,
                                   const uint8_t* mk, Pre pre, Fin fin) {
    using H = Halo<R>;
    constexpr int S = 2 * R + 1;
    int off[H::NF];
#pragma unroll
    for (int it = 0; it < H::NF; ++it) {
        const int i = threadIdx.x + it * kBlock;
        const int yy = by * kTY - R + i / H::HX, xx = bx * kTX - R + i % H::HX;
        const bool in = i < H::NI && xx >= 0 && xx < P.n[0] && yy >= 0 && yy < P.n[1];
        off[it] = in ? 4 * (yy * P.n[0] + xx) : kNoElem;
    }
    double ring[S][NCH];
    double zs[NCH];
#pragma unroll
    for (int k = 0; k < S; ++k)
#pragma unroll
        for (int c = 0; c < NCH; ++c) ring[k][c] = 0.0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) zs[c] = 0.0;
    const int zlast = z1 - 1 + R;
    TileRegs<R> t;
    fetch_tile<R, MODE>(P, off, z0 - R, a0, a1, a2, mk, t);
    commit_tile<R, NCH, MODE>(L[0], t);
    fetch_tile<R, MODE>(P, off, z0 - R + 1, a0, a1, a2, mk, t);
    __syncthreads();
    int b = 0, zz = z0 - R;
    // one plane; k (a constant: #pragma unroll gives up on nine of these
    // bodies, and the ring would move to scratch) is its ring slot
    const auto step = [&](auto slot) __attribute__((always_inline)) {
        constexpr int k = decltype(slot)::value;
        if (zz > zlast) return;  // uniform over the block
        x_sums<R, NCH, MODE>(L[b]);
        commit_tile<R, NCH, MODE>(L[b ^ 1], t);   // plane zz + 1
        fetch_tile<R, MODE>(P, off, zz + 2, a0, a1, a2, mk, t);
        __syncthreads();
        double p[NCH], s[NCH];
        y_sums<R, NCH>(L[b], p);
        b ^= 1;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            zs[c] += p[c] - ring[k][c];   // ring[k] holds plane zz - S, leaving now
            ring[k][c] = p[c];
        }
        own_row<NCH>(zs, s);
        fin(zz - R, s);   // its window [z - R, z + R] is complete
        pre(zz - R + 1);
        ++zz;
    };
    while (zz <= zlast) for_slots(step, std::make_integer_sequence<int, S>());
}

template <int R>
__global__ void __launch_bounds__(kBlock, 2)
k_lcc_stats_fused(const PairDesc P, int zc, const float* __restrict__ F, const float* __restrict__ W,
                  const uint8_t* __restrict__ mk, float* __restrict__ A, double* __restrict__ part) {
    __shared__ XYPlane<R, 6> L[2];
    __shared__ double red[2 * (kBlock / 64)];
    const int ntx = cdiv(P.n[0], kTX), nty = cdiv(P.n[1], kTY);
    const int item = xcd_item(blockIdx.x, ntx * nty * cdiv(P.n[2], zc), 0);
    if (item < 0) return;
    const int bx = item % ntx, by = (item / ntx) % nty;
    const int z0 = (item / (ntx * nty)) * zc, z1 = min(P.n[2], z0 + zc);
    const int x = bx * kTX + threadIdx.x % kTX, y = by * kTY + threadIdx.x / kTX;
    const bool col = x < P.n[0] && y < P.n[1];
    const uint32_t N = (uint32_t)P.nvox;
    const int c0 = col ? y * P.n[0] + x : kNoElem, c4 = col ? 4 * c0 : kNoElem;
    const int sz = P.n[0] * P.n[1];
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(mk, N);
    const __amdgpu_buffer_rsrc_t rB = make_rsrc(A, 4 * N), rD = make_rsrc(A + P.nvox, 4 * N),
                                 rE = make_rsrc(A + 2 * P.nvox, 4 * N);
    double acc[2] = {0.0, 0.0};
    uint8_t mnext = 0;
    z_ring_walk<R, 6, 0>(
        P, L, bx, by, z0, z1, F, W, nullptr, mk,
        [&](int z) {
            const bool on = z >= z0 && z < z1;
            mnext = load1u8(rm, on ? c0 : kNoElem, on ? z * sz : 0);
        },
        [&](int z, const double* s) {
            float aB = 0.f, aD = 0.f, aE = 0.f;
            if (mnext) {
                double rho;
                lcc_coef(s, &aB, &aD, &aE, &rho);
                acc[0] += 1.0;
                acc[1] += rho;
            }
            const int vo = z >= z0 ? c4 : kNoElem, so = z >= z0 ? 4 * z * sz : 0;
            store1(rB, aB, vo, so);
            store1(rD, aD, vo, so);
            store1(rE, aE, vo, so);
        });
    block_sum<kBlock, 2>(acc, red);
    if (threadIdx.x == 0) {
        part[2 * item] = acc[0];
        part[2 * item + 1] = acc[1];
    }
}

template <int R, int DIM>
__global__ void __launch_bounds__(kBlock)
k_lcc_grad_fused(const PairDesc P, int zc, const float* __restrict__ A, const float* __restrict__ F,
                 const float* __restrict__ W, const uint8_t* __restrict__ mk,
                 const float* __restrict__ dW, const double* __restrict__ scal, float lambda,
                 int lam_acc, float* __restrict__ g) {
    __shared__ XYPlane<R, 3> L[2];
    const int ntx = cdiv(P.n[0], kTX), nty = cdiv(P.n[1], kTY);
    const int item = xcd_item(blockIdx.x, ntx * nty * cdiv(P.n[2], zc), 0);
    if (item < 0) return;
    const int bx = item % ntx, by = (item / ntx) % nty;
    const int z0 = (item / (ntx * nty)) * zc, z1 = min(P.n[2], z0 + zc);
    const int x = bx * kTX + threadIdx.x % kTX, y = by * kTY + threadIdx.x / kTX;
    const bool col = x < P.n[0] && y < P.n[1];
    const long long N = P.nvox;
    const uint32_t nb = 4u * (uint32_t)N;
    const int c0 = col ? y * P.n[0] + x : kNoElem, c4 = col ? 4 * c0 : kNoElem;
    const int sz = P.n[0] * P.n[1];
    const double inv = scal[0];
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(mk, (uint32_t)N), rw = make_rsrc(W, nb),
                                 rf = make_rsrc(F, nb);
    __amdgpu_buffer_rsrc_t rd[DIM], rg[DIM], rg0[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        rd[a] = make_rsrc(dW + a * N, nb);
        rg[a] = make_rsrc(g + a * N, nb);
        rg0[a] = make_rsrc(g + a * N, lam_acc ? nb : 0u);   // zeros where nothing is added to
    }
    // per-voxel inputs of the next output plane
    uint8_t m = 0;
    float w = 0.f, f = 0.f, d[DIM], g0[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) d[a] = g0[a] = 0.f;
    z_ring_walk<R, 3, 1>(
        P, L, bx, by, z0, z1, A, A + N, A + 2 * N, nullptr,
        [&](int z) {
            const bool on = z >= z0 && z < z1;
            const int vo = on ? c4 : kNoElem, so = on ? 4 * z * sz : 0;
            m = load1u8(rm, on ? c0 : kNoElem, on ? z * sz : 0);
            w = load1(rw, vo, so);
            f = load1(rf, vo, so);
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                d[a] = load1(rd[a], vo, so);
                g0[a] = load1(rg0[a], vo, so);
            }
        },
        [&](int z, const double* s) {
            const float t = (float)(-inv * (s[0] + 2.0 * (double)w * s[1] + (double)f * s[2]));
            const float dsdw = m ? t : 0.f;
            const int vo = z >= z0 ? c4 : kNoElem, so = z >= z0 ? 4 * z * sz : 0;
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                const float img = dsdw * d[a] * P.s[a];
                store1(rg[a], lam_acc ? fmaf(lambda, g0[a], img) : img, vo, so);
            }
        });
}

__host__ inline int fused_tiles(const PairDesc& P) {
    return cdiv(P.n[0], kTX) * cdiv(P.n[1], kTY);
}

// Output planes per block of the fused passes: a CU runs its blocks' zc + 2r
// planes at a fixed rate, so the launch takes about ceil(blocks / 256) (zc +
// 2r) plane steps, and 1.45 where a CU has a single block (nothing hides its
// latency). The even split of z that takes the fewest is used, of kMinZc to
// kMaxZc planes. Whole evaluations, the rule against 16 planes always: 87 x 152
// x 89 (r 3) 120 and 131 us, 77 x 85 x 119 (r 2) 93 and 109, 111 x 77 x 158 (r 4)
// 136 and 141, 64^3 (r 3) 76 and 100; 128^3 has 16 from the rule (the same
// inputs over and over: 136 us; 8 planes 150, 32 151).
constexpr int kMinZc = 4, kMaxZc = 64;
__host__ inline int fused_zc(const PairDesc& P, int r) {
    const int tiles = fused_tiles(P), nz = P.n[2];
    long long best = 0;
    int zc = 0;
    for (int m = min(nz, kMaxZc); m >= min(nz, kMinZc); --m) {
        const int k = cdiv(nz, m), c = cdiv(nz, k);
        const long long per_cu = ((long long)tiles * k + 255) / 256;
        const long long cost = (per_cu == 1 ? 29 : 20 * per_cu) * (c + 2 * r);
        if (!zc || cost < best) {
            best = cost;
            zc = c;
        }
    }
    return zc;
}

__host__ inline size_t box_lds(int nch, int r) {
    const int HX = kTX + 2 * r, HY = kTY + 2 * r;
    return sizeof(double) * ((3 * HY * HX + 1) / 2 + (size_t)nch * HY * kTX);
}

}  // namespace

// Whether the fused passes (no FP64 box-sum maps) serve this dimension and radius.
bool lcc_fused(int dim, int r) { return dim == 3 && r >= 1 && r <= kMaxFusedR; }

// Partial-sum slots of the statistics pass (the larger of the two forms).
int lcc_partials(const PairDesc& P, int dim, int r) {
    const long long items = (long long)P.n[0] * P.n[1] * cdiv(P.n[2], kZSeg);
    const int zpass = (int)((items + kBlock - 1) / kBlock);
    return lcc_fused(dim, r) ? fused_tiles(P) * cdiv(P.n[2], fused_zc(P, r)) : zpass;
}

// LDS of the box passes at radius r (the largest, six channels).
size_t lcc_lds_bytes(int r) { return box_lds(6, r); }

// S (and, with grad, dS/du) of the LCC at displacement u. Buffers: W, dW
// ([d][N]) float; mk uint8 [N]; S double [6][N]; A float [3][N]; part double
// [2 * lcc_partials]; scal double [1]. value: S, or S + lambda * value when
// lam_acc (the regulariser written there before); grad: dS/du, or
// dS/du + lambda * grad when lam_acc.
hipError_t launch_lcc(const PairDesc& P, int dim, int r, const float* F, const float* M,
                      const float* u, float* Wb, uint8_t* mk, float* dW, double* S, float* A,
                      double* part, double* scal, uint32_t* flag, float lambda, bool lam_acc,
                      float* value, float* grad, hipStream_t s) {
    const int rz = dim == 3 ? r : 0;
    const int nxy = cdiv(P.n[0], kTX) * cdiv(P.n[1], kTY) * P.n[2];
    const int acc = lam_acc ? 1 : 0;
    const int ns = xcd_grid(cdiv(P.n[0] * P.n[1], kBlock) * cdiv(P.n[2], kSampleZ), 0);
    if (dim == 3)
        hipLaunchKernelGGL(k_lcc_sample<3>, dim3(ns), dim3(kBlock), 0, s, P, M, u,
                           Wb, mk, dW);
    else
        hipLaunchKernelGGL(k_lcc_sample<2>, dim3(ns), dim3(kBlock), 0, s, P, M, u,
                           Wb, mk, dW);
    if (lcc_fused(dim, r)) {
        // fused passes: no FP64 maps in memory
        const int zc = fused_zc(P, r), nb = fused_tiles(P) * cdiv(P.n[2], zc);
        const int nblk = xcd_grid(nb, 0);
        switch (r) {
            case 1:
                hipLaunchKernelGGL(k_lcc_stats_fused<1>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wb, mk, A, part);
                break;
            case 2:
                hipLaunchKernelGGL(k_lcc_stats_fused<2>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wb, mk, A, part);
                break;
            case 3:
                hipLaunchKernelGGL(k_lcc_stats_fused<3>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wb, mk, A, part);
                break;
            default:
                hipLaunchKernelGGL(k_lcc_stats_fused<4>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wb, mk, A, part);
                break;
        }
        hipLaunchKernelGGL(k_lcc_value, dim3(1), dim3(kBlock), 0, s, part, nb, lambda, acc, value,
                           scal, flag);
        if (!grad) return hipGetLastError();
        switch (r) {
            case 1:
                hipLaunchKernelGGL((k_lcc_grad_fused<1, 3>), dim3(nblk), dim3(kBlock), 0, s, P, zc, A,
                                   F, Wb, mk, dW, scal, lambda, acc, grad);
                break;
            case 2:
                hipLaunchKernelGGL((k_lcc_grad_fused<2, 3>), dim3(nblk), dim3(kBlock), 0, s, P, zc, A,
                                   F, Wb, mk, dW, scal, lambda, acc, grad);
                break;
            case 3:
                hipLaunchKernelGGL((k_lcc_grad_fused<3, 3>), dim3(nblk), dim3(kBlock), 0, s, P, zc, A,
                                   F, Wb, mk, dW, scal, lambda, acc, grad);
                break;
            default:
                hipLaunchKernelGGL((k_lcc_grad_fused<4, 3>), dim3(nblk), dim3(kBlock), 0, s, P, zc, A,
                                   F, Wb, mk, dW, scal, lambda, acc, grad);
                break;
        }
        return hipGetLastError();
    }
    const int nblk = (int)(((long long)P.n[0] * P.n[1] * cdiv(P.n[2], kZSeg) + kBlock - 1) / kBlock);
    hipLaunchKernelGGL((k_lcc_box_xy<6, 0>), dim3(nxy), dim3(kBlock), box_lds(6, r), s, P, r, F,
                       Wb, nullptr, mk, S);
    hipLaunchKernelGGL(k_lcc_stats_z, dim3(nblk), dim3(kBlock), 0, s, P, rz, S, F, Wb, mk, A,
                       part);
    hipLaunchKernelGGL(k_lcc_value, dim3(1), dim3(kBlock), 0, s, part, nblk, lambda, acc, value,
                       scal, flag);
    if (!grad) return hipGetLastError();
    // the coefficient box sums reuse the statistics buffer
    hipLaunchKernelGGL((k_lcc_box_xy<3, 1>), dim3(nxy), dim3(kBlock), box_lds(3, r), s, P, r, A,
                       A + P.nvox, A + 2 * P.nvox, mk, S);
    if (dim == 3)
        hipLaunchKernelGGL(k_lcc_grad_z<3>, dim3(nblk), dim3(kBlock), 0, s, P, rz, S, F, Wb, mk,
                           dW, scal, lambda, acc, grad);
    else
        hipLaunchKernelGGL(k_lcc_grad_z<2>, dim3(nblk), dim3(kBlock), 0, s, P, rz, S, F, Wb, mk,
                           dW, scal, lambda, acc, grad);
    return hipGetLastError();
}

// S of the LCC for a given warped image and mask (no gradient).
hipError_t launch_lcc_value(const PairDesc& P, int dim, int r, const float* F, const float* Wimg,
                            const uint8_t* mk, double* S, float* A, double* part, double* scal,
                            uint32_t* flag, float* value, hipStream_t s) {
    const int rz = dim == 3 ? r : 0;
    const int nxy = cdiv(P.n[0], kTX) * cdiv(P.n[1], kTY) * P.n[2];
    if (lcc_fused(dim, r)) {
        const int zc = fused_zc(P, r), nb = fused_tiles(P) * cdiv(P.n[2], zc);
        const int nblk = xcd_grid(nb, 0);
        switch (r) {
            case 1:
                hipLaunchKernelGGL(k_lcc_stats_fused<1>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wimg, mk, A, part);
                break;
            case 2:
                hipLaunchKernelGGL(k_lcc_stats_fused<2>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wimg, mk, A, part);
                break;
            case 3:
                hipLaunchKernelGGL(k_lcc_stats_fused<3>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wimg, mk, A, part);
                break;
            default:
                hipLaunchKernelGGL(k_lcc_stats_fused<4>, dim3(nblk), dim3(kBlock), 0, s, P, zc, F,
                                   Wimg, mk, A, part);
                break;
        }
        hipLaunchKernelGGL(k_lcc_value, dim3(1), dim3(kBlock), 0, s, part, nb, 0.f, 0, value, scal,
                           flag);
        return hipGetLastError();
    }
    const int nblk = (int)(((long long)P.n[0] * P.n[1] * cdiv(P.n[2], kZSeg) + kBlock - 1) / kBlock);
    hipLaunchKernelGGL((k_lcc_box_xy<6, 0>), dim3(nxy), dim3(kBlock), box_lds(6, r), s, P, r, F,
                       Wimg, nullptr, mk, S);
    hipLaunchKernelGGL(k_lcc_stats_z, dim3(nblk), dim3(kBlock), 0, s, P, rz, S, F, Wimg, mk, A,
                       part);
    hipLaunchKernelGGL(k_lcc_value, dim3(1), dim3(kBlock), 0, s, part, nblk, 0.f, 0, value, scal,
                       flag);
    return hipGetLastError();
}

}  // namespace air

// this unit's bounds-check flags (debug build only)
AIR_DEBUG_UNIT(lcc)
