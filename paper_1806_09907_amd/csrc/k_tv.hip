// Total-variation regularisers (Sec. III-F) on a dense displacement u:
//   anisotropic: R = (1/|X_R|) sum_{x in X_R} sum_c sum_a |D_a u_c(x)|
//   isotropic:   R = (1/|X_R|) sum_{x in X_R} sqrt(sum_c sum_a D_a u_c(x)^2)
// with the forward differences D_a u_c(x) = u_c(x + e_a) - u_c(x) over
// X_R = prod_a [0, n_a - 2] (the diffusion term's discretisation) and the
// subgradient 0 where a term is 0. Every voxel x gets
//   dR/du_c(x) = (1/|X_R|) (sum_a [x - e_a in X_R] k_ca(x - e_a)
//                           - [x in X_R] sum_a k_ca(x)),
// k = sign(D) (anisotropic) or D / ||J|| (isotropic), where J(y) is the
// matrix of differences at y. The Gram form of the diffusion term has no TV
// counterpart, so a B-spline field is expanded to the voxel grid first.
#include "device_common.h"

namespace air {

namespace {

constexpr int kTvBlocks = 4096;
// items: kBlock columns by zc planes
__host__ __device__ inline int tv_items(const PairDesc& P, int zc) {
    return cdiv(P.n[0] * P.n[1], kBlock) * cdiv(P.n[2], zc);
}
// Planes a thread walks: 8, or fewer where that leaves less than two blocks
// a CU (a walk's planes are a serial chain of loads): 48 x 40 x 33
// takes 32.7 us an evaluation so and 37.5 with 8, 64^3 57.6 and 61.4.
__host__ inline int tv_zc(const PairDesc& P) {
    int zc = 8;
    while (zc > 1 && tv_items(P, zc) < 512) zc /= 2;
    return zc;
}

// k_ca for every c, a from the differences at a point of X_R; returns the
// term's value there.
template <int DIM, int KIND>
__device__ inline float tv_coef(const float (*D)[3], float (*k)[3]) {
    float ss = 0.f, l1 = 0.f;
#pragma unroll
    for (int c = 0; c < DIM; ++c)
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            ss += D[c][a] * D[c][a];
            l1 += fabsf(D[c][a]);
        }
    if (KIND == AIR_REG_ANISO_TV) {
#pragma unroll
        for (int c = 0; c < DIM; ++c)
#pragma unroll
            for (int a = 0; a < DIM; ++a)
                k[c][a] = D[c][a] > 0.f ? 1.f : (D[c][a] < 0.f ? -1.f : 0.f);
        return l1;
    }
    const float nrm = sqrtf(ss);
    const float inv = nrm > 0.f ? 1.f / nrm : 0.f;
#pragma unroll
    for (int c = 0; c < DIM; ++c)
#pragma unroll
        for (int a = 0; a < DIM; ++a) k[c][a] = D[c][a] * inv;
    return nrm;
}

// What a plane adds to the values a column carries: the neighbours of the
// voxel within its plane, the three points of the plane above that the terms
// at x, x - e_x and x - e_y reach, and the gradient to add to.
template <int DIM>
struct TvRow {
    float xp[DIM], yp[DIM], xmyp[DIM], xpym[DIM], u1[DIM], xm1[DIM], ym1[DIM], g[DIM];
};

// grad (+)= scale * dR/du; partial[block] = sum over the block's voxels in X_R
// of the term (FP64). Bound by its loads: a voxel's gradient needs the terms
// at four points, 48 values when each is formed by itself. A thread walks
// zc planes of one column: the three values of the plane above are the next
// plane's own, and its term at x - e_z is the last plane's term at x, so a
// voxel loads 21 values, one plane ahead of their use; neighbouring items run
// on one XCD. 128^3 (anisotropic, added to a gradient): 20.9 -> 18.4 us;
// whole evaluations 181 x 217 x 181 isotropic 244 -> 196 us, 256^3 664 -> 583.
template <int DIM, int KIND>
__global__ void __launch_bounds__(kBlock)
k_tv(const PairDesc P, int zc, const float* __restrict__ u, float scale, float* __restrict__ grad,
     int accumulate, double* __restrict__ partial) {
    __shared__ double red[8 * (kBlock / 64)];
    const long long N = P.nvox;
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2], sz = nx * ny;
    const int ncb = cdiv(sz, kBlock), T = tv_items(P, zc), tq = (T + 7) / 8;
    const float inv_xr = P.inv_xr;
    const uint32_t nb = 4u * (uint32_t)N;
    __amdgpu_buffer_rsrc_t ru[DIM], rg[DIM], rg0[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        ru[c] = make_rsrc(u + c * N, nb);
        rg[c] = make_rsrc(grad + c * N, nb);
        rg0[c] = make_rsrc(grad + c * N, accumulate ? nb : 0u);
    }
    double acc[1] = {0.0};
    // the items of XCD b % 8 are one contiguous run
    for (int i = blockIdx.x / 8; i < tq; i += gridDim.x / 8) {
        const int item = blockIdx.x % 8 * tq + i;
        if (item >= T) break;
        const int z0 = item / ncb * zc, z1 = min(nz, z0 + zc);
        const int col = (item % ncb) * kBlock + threadIdx.x;
        const bool on = col < sz;
        const int y = col / nx, x = col - y * nx;
        const bool xr = on && x <= nx - 2, yr = on && y <= ny - 2, xl = on && x >= 1,
                   yl = on && y >= 1;
        const int o0 = on ? 4 * col : kNoElem, oxp = xr ? 4 * (col + 1) : kNoElem,
                  oyp = yr ? 4 * (col + nx) : kNoElem, oxm = xl ? 4 * (col - 1) : kNoElem,
                  oym = yl ? 4 * (col - nx) : kNoElem,
                  oxmyp = xl && yr ? 4 * (col - 1 + nx) : kNoElem,
                  oxpym = xr && yl ? 4 * (col + 1 - nx) : kNoElem;
        const auto fetch = [&](int z, TvRow<DIM>& r) {
            const bool zi = z < z1;
            const int so = zi ? 4 * z * sz : 0;
            // the plane above, where there is one
            const bool up = DIM == 3 && zi && z + 1 < nz;
            const int so1 = up ? 4 * (z + 1) * sz : 0;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                r.xp[c] = load1(ru[c], zi ? oxp : kNoElem, so);
                r.yp[c] = load1(ru[c], zi ? oyp : kNoElem, so);
                r.xmyp[c] = load1(ru[c], zi ? oxmyp : kNoElem, so);
                r.xpym[c] = load1(ru[c], zi ? oxpym : kNoElem, so);
                if (DIM == 3) {
                    r.u1[c] = load1(ru[c], up ? o0 : kNoElem, so1);
                    r.xm1[c] = load1(ru[c], up ? oxm : kNoElem, so1);
                    r.ym1[c] = load1(ru[c], up ? oym : kNoElem, so1);
                }
                r.g[c] = load1(rg0[c], zi ? o0 : kNoElem, so);
            }
        };
        TvRow<DIM> r;
        fetch(z0, r);
        float u0[DIM], xm[DIM], ym[DIM], kz[DIM];
        float D[3][3], k[3][3];
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            u0[c] = load1(ru[c], o0, 4 * z0 * sz);
            xm[c] = load1(ru[c], oxm, 4 * z0 * sz);
            ym[c] = load1(ru[c], oym, 4 * z0 * sz);
            kz[c] = 0.f;
        }
        if (DIM == 3 && z0 > 0) {   // the term at z0 - 1
            const int so = 4 * (z0 - 1) * sz;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                const float b = load1(ru[c], o0, so);
                D[c][0] = load1(ru[c], oxp, so) - b;
                D[c][1] = load1(ru[c], oyp, so) - b;
                D[c][2] = u0[c] - b;
            }
            tv_coef<DIM, KIND>(D, k);
#pragma unroll
            for (int c = 0; c < DIM; ++c) kz[c] = xr && yr ? k[c][2] : 0.f;
        }
        for (int z = z0; z < z1; ++z) {
            TvRow<DIM> t = r;
            fetch(z + 1, r);
            const bool zr = DIM == 2 || z <= nz - 2;
            float g[DIM];
            // the term at x
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                D[c][0] = t.xp[c] - u0[c];
                D[c][1] = t.yp[c] - u0[c];
                if (DIM == 3) D[c][2] = t.u1[c] - u0[c];
            }
            const float val = tv_coef<DIM, KIND>(D, k);
            const bool in_r = xr && yr && zr;
            acc[0] += in_r ? (double)val : 0.0;
            float kn[DIM];
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                g[c] = 0.f;
#pragma unroll
                for (int a = 0; a < DIM; ++a) g[c] -= k[c][a];
                g[c] = in_r ? g[c] : 0.f;
                kn[c] = in_r && DIM == 3 ? k[c][2] : 0.f;
            }
            // at x - e_x
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                D[c][0] = u0[c] - xm[c];
                D[c][1] = t.xmyp[c] - xm[c];
                if (DIM == 3) D[c][2] = t.xm1[c] - xm[c];
            }
            tv_coef<DIM, KIND>(D, k);
#pragma unroll
            for (int c = 0; c < DIM; ++c) g[c] += xl && yr && zr ? k[c][0] : 0.f;
            // at x - e_y
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                D[c][0] = t.xpym[c] - ym[c];
                D[c][1] = u0[c] - ym[c];
                if (DIM == 3) D[c][2] = t.ym1[c] - ym[c];
            }
            tv_coef<DIM, KIND>(D, k);
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                g[c] += xr && yl && zr ? k[c][1] : 0.f;
                g[c] += kz[c];   // at x - e_z
                const float v = scale * inv_xr * g[c];
                store1(rg[c], accumulate ? t.g[c] + v : v, o0, 4 * z * sz);
                if (DIM == 3) {
                    u0[c] = t.u1[c];
                    xm[c] = t.xm1[c];
                    ym[c] = t.ym1[c];
                    kz[c] = kn[c];
                }
            }
        }
    }
    block_sum<kBlock, 1>(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc[0];
}

// *value (+)= weight * (sum of the partials) / |X_R|, in block order.
__global__ void __launch_bounds__(kBlock)
k_tv_value(const double* __restrict__ partial, int nblk, float inv_xr, float weight, float* value,
           int accumulate) {
    __shared__ double red[8 * (kBlock / 64)];
    double s[1] = {0.0};
    for (int b = threadIdx.x; b < nblk; b += kBlock) s[0] += partial[b];
    block_sum<kBlock, 1>(s, red);
    if (threadIdx.x == 0) {
        const float r = (float)((double)weight * s[0] * (double)inv_xr);
        *value = accumulate ? *value + r : r;
    }
}

}  // namespace

// grad (+)= scale * dR/du and *value (+)= weight * R for the plan's TV kind.
// partial: at least tv_partials() doubles of workspace.
int tv_partials() { return kTvBlocks; }

hipError_t launch_tv(const PairDesc& P, int dim, int kind, const float* u, float scale,
                     float* grad, bool accumulate_grad, double* partial, float weight,
                     float* value, bool accumulate_value, hipStream_t s) {
    const int zc = tv_zc(P), g = min(xcd_grid(tv_items(P, zc), 0), kTvBlocks);
    const int acc = accumulate_grad ? 1 : 0;
    if (dim == 3) {
        if (kind == AIR_REG_ANISO_TV)
            hipLaunchKernelGGL((k_tv<3, AIR_REG_ANISO_TV>), dim3(g), dim3(kBlock), 0, s, P, zc,
                               u, scale, grad, acc, partial);
        else
            hipLaunchKernelGGL((k_tv<3, AIR_REG_ISO_TV>), dim3(g), dim3(kBlock), 0, s, P, zc,
                               u, scale, grad, acc, partial);
    } else {
        if (kind == AIR_REG_ANISO_TV)
            hipLaunchKernelGGL((k_tv<2, AIR_REG_ANISO_TV>), dim3(g), dim3(kBlock), 0, s, P, zc,
                               u, scale, grad, acc, partial);
        else
            hipLaunchKernelGGL((k_tv<2, AIR_REG_ISO_TV>), dim3(g), dim3(kBlock), 0, s, P, zc,
                               u, scale, grad, acc, partial);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tv_value, dim3(1), dim3(kBlock), 0, s, partial, g, P.inv_xr, weight,
                       value, accumulate_value ? 1 : 0);
    return hipGetLastError();
}

}  // namespace air
