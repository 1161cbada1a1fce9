// Vector kernels of the Krylov solver and the interface loop (double).
//
// Reductions are deterministic: a fixed grid of kRedBlocks blocks writes one
// partial per block (wave shuffles, then LDS in a fixed order) and a single
// block adds the partials in a fixed order.  Results are bitwise
// reproducible from run to run.
#include <utility>

#include "internal.h"

namespace sdbie {
namespace {


// block of 256 lanes -> sum in lane 0 (fixed order)
__device__ __forceinline__ double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return r;
}

// The reductions over kRedBlocks blocks launch only those that hold elements
// (len / 256 of them, red_blocks); the first clears the others' partials.
__device__ __forceinline__ void clear_partials(double* __restrict__ part) {
    if (blockIdx.x == 0)
        for (int b = gridDim.x + threadIdx.x; b < kRedBlocks; b += 256) part[b] = 0.0;
}
inline unsigned red_blocks(int64_t len) {
    return len < (int64_t)kRedBlocks * 256 ? (unsigned)((len + 255) / 256) : (unsigned)kRedBlocks;
}

__global__ __launch_bounds__(256) void k_dot_partial(const double* __restrict__ a, const double* __restrict__ b,
                                                     int64_t len, double* __restrict__ part) {
    __shared__ double sh[4];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (int64_t)kRedBlocks * 256)
        s += b ? a[i] * b[i] : a[i];
    const double r = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
    clear_partials(part);
}

// part: [k][nb] -> out[j] = sum_b part[j][b], one block per j
__global__ __launch_bounds__(256) void k_reduce_cols(const double* __restrict__ part, int nb,
                                                     double* __restrict__ out) {
    __shared__ double sh[4];
    const int j = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) s += part[(int64_t)j * nb + b];
    const double r = block_sum(s, sh);
    if (threadIdx.x == 0) out[j] = r;
}

// part[j][b] = sum over block b's chunk of V_j . w; blockIdx.y takes kDotCols
// columns at a time, so w is read once per kDotCols columns (fixed order)
constexpr int kDotCols = 8;
__global__ __launch_bounds__(256) void k_multidot_partial(const double* __restrict__ V, int64_t ld, int k,
                                                          const double* __restrict__ w, int64_t len,
                                                          double* __restrict__ part) {
    __shared__ double sh[4];
    const int64_t chunk = (len + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < len ? lo + chunk : len;
    const int j0 = blockIdx.y * kDotCols;
    const int nc = k - j0 < kDotCols ? k - j0 : kDotCols;
    double acc[kDotCols];
#pragma unroll
    for (int c = 0; c < kDotCols; ++c) acc[c] = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const double wi = w[i];
#pragma unroll
        for (int c = 0; c < kDotCols; ++c)
            if (c < nc) acc[c] += V[(int64_t)(j0 + c) * ld + i] * wi;
    }
    for (int c = 0; c < nc; ++c) {
        const double r = block_sum(acc[c], sh);
        if (threadIdx.x == 0) part[(int64_t)(j0 + c) * gridDim.x + blockIdx.x] = r;
    }
}

// the same for chunks of at most 64 elements: a wave per chunk (the block's other
// waves would add zeros), 128 blocks instead of 512
__global__ __launch_bounds__(256) void k_multidot_small(const double* __restrict__ V, int64_t ld, int k,
                                                        const double* __restrict__ w, int64_t len,
                                                        double* __restrict__ part) {
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t chunk = (len + kRedBlocks - 1) / kRedBlocks, i = b * chunk + lane;
    const bool in = lane < chunk && i < len;
    const double wi = in ? w[i] : 0.0;
    const int j0 = blockIdx.y * kDotCols;
    const int nc = k - j0 < kDotCols ? k - j0 : kDotCols;
    for (int c = 0; c < nc; ++c) {
        const double r = wave_sum(in ? V[(int64_t)(j0 + c) * ld + i] * wi : 0.0);
        if (lane == 0) part[(int64_t)(j0 + c) * kRedBlocks + b] = r;
    }
}

// ---- fused Gram-Schmidt ------------------------------------------------------
// One Krylov step orthogonalises w against k columns twice and normalises it.
// As separate kernels that is nine launches, most of them a few microseconds of
// launch and drain around less work (n = 2650: 45 us of a 250 us iteration).
// Here each kernel reduces the previous one's block partials itself (every block
// redundantly: k columns of 512 partials from L2) and ends on the partials of the
// next dot products: k_multidot_partial, k_cgs_step, k_cgs_last, k_cgs_scale.
// The additions are those of k_reduce_cols, k_multi_axpy, k_multidot_partial and
// k_dot_partial in their order, so the results are the same bit for bit.

// sum of kRedBlocks block partials by one wave: k_reduce_cols' order (its four
// waves' trees, then (0 + 1) + (2 + 3))
__device__ __forceinline__ double reduce_blocks(const double* __restrict__ part) {
    const int lane = threadIdx.x & 63;
    static_assert(kRedBlocks == 512, "two partials per thread of a 256-thread block");
    double r[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = wave_sum(part[64 * v + lane] + part[64 * v + lane + 256]);
    return (r[0] + r[1]) + (r[2] + r[3]);
}

// h[j] = sum of column j's partials, j < k (k <= kFuseCols); ends on a barrier
__device__ __forceinline__ void reduce_columns(const double* __restrict__ part, int k, double* h) {
    for (int j = threadIdx.x >> 6; j < k; j += 4) {
        const double r = reduce_blocks(part + (int64_t)j * kRedBlocks);
        if ((threadIdx.x & 63) == 0) h[j] = r;
    }
    __syncthreads();
}

// a b + c d with each product rounded (what the host computes; fma would not be)
__device__ __forceinline__ double two_products(double a, double b, double c, double d) {
#pragma clang fp contract(off)
    const double x = a * b, y = c * d;
    return x + y;
}

// w -= Vs h with h from part_in, on block b's chunk; then the partials of Vd . w.
// With rot (the Givens rotations c[0..ks-1), s[0..ks-1) of a deflation space), h
// is turned into e = Q^T h and the subtracted vector is V (Q e): what the host
// did between two copies, unfused multiplies and adds as there.
// Block 0 writes h (with rot: e) to hout, host memory.
// SMALL: chunks of at most 64 elements, a wave per chunk (as k_multidot_small):
// the columns are then reduced by 128 blocks, not 512.
template <bool SMALL>
__global__ __launch_bounds__(256) void k_cgs_step(const double* __restrict__ Vs, int64_t lds, int ks,
                                                  const double* __restrict__ part_in, const double* __restrict__ rot,
                                                  double* __restrict__ hout, const double* __restrict__ Vd,
                                                  int64_t ldd, int kd, double* w, int64_t len,
                                                  double* __restrict__ part_out) {
    __shared__ double h[kFuseCols], sc[2 * kFuseCols], sh[kDotCols][4];
    const int tid = threadIdx.x;
    if (rot)
        for (int j = tid; j < 2 * (ks - 1); j += 256) sc[j] = rot[j];
    reduce_columns(part_in, ks, h);
    if (rot) {
        const int kr = ks - 1;
        if (tid == 0) {
            const double *c = sc, *sn = sc + kr;
            double cur = h[0];
#pragma unroll 4
            for (int j = 0; j < kr; ++j) {
                const double nxt = h[j + 1];
                h[j] = two_products(c[j], cur, sn[j], nxt);
                cur = two_products(-sn[j], cur, c[j], nxt);
            }
            if (blockIdx.x == 0)
                for (int j = 0; j < kr; ++j) hout[j] = h[j];
            cur = 0.0;
#pragma unroll 4
            for (int j = kr - 1; j >= 0; --j) {
                const double g = h[j];
                h[j + 1] = two_products(sn[j], g, c[j], cur);
                cur = two_products(c[j], g, -sn[j], cur);
            }
            h[0] = cur;
        }
        __syncthreads();
    } else if (blockIdx.x == 0 && tid < ks) {
        hout[tid] = h[tid];
    }
    const int64_t chunk = (len + kRedBlocks - 1) / kRedBlocks;
    if constexpr (SMALL) {
        const int b = blockIdx.x * 4 + (tid >> 6), lane = tid & 63;
        const int64_t i = b * chunk + lane;
        const bool in = lane < chunk && i < len;
        double wi = 0.0;
        if (in) {
            double s = 0.0;
#pragma unroll 4
            for (int j = 0; j < ks; ++j) s = fma(h[j], Vs[(int64_t)j * lds + i], s);
            wi = w[i] - s;
            w[i] = wi;
        }
#pragma unroll 4
        for (int j = 0; j < kd; ++j) {
            const double r = wave_sum(in ? Vd[(int64_t)j * ldd + i] * wi : 0.0);
            if (lane == 0) part_out[(int64_t)j * kRedBlocks + b] = r;
        }
        return;
    }
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < len ? lo + chunk : len;
    for (int64_t i = lo + tid; i < hi; i += 256) {
        double s = 0.0;
        for (int j = 0; j < ks; ++j) s = fma(h[j], Vs[(int64_t)j * lds + i], s);
        w[i] -= s;
    }
    for (int j0 = 0; j0 < kd; j0 += kDotCols) {
        const int nc = kd - j0 < kDotCols ? kd - j0 : kDotCols;
        double acc[kDotCols];
#pragma unroll
        for (int c = 0; c < kDotCols; ++c) acc[c] = 0.0;
        for (int64_t i = lo + tid; i < hi; i += 256) {
            const double wi = w[i];
#pragma unroll
            for (int c = 0; c < kDotCols; ++c)
                if (c < nc) acc[c] = fma(Vd[(int64_t)(j0 + c) * ldd + i], wi, acc[c]);
        }
#pragma unroll
        for (int c = 0; c < kDotCols; ++c) {
            const double r = wave_sum(acc[c]);
            if ((tid & 63) == 0) sh[c][tid >> 6] = r;
        }
        __syncthreads();
        if (tid < nc)
            part_out[(int64_t)(j0 + tid) * kRedBlocks + blockIdx.x] =
                (sh[tid][0] + sh[tid][1]) + (sh[tid][2] + sh[tid][3]);
        __syncthreads();
    }
}

// w -= V h with h from part_in; then the partials of w . w
__global__ __launch_bounds__(256) void k_cgs_last(const double* __restrict__ V, int64_t ld, int k,
                                                  const double* __restrict__ part_in, double* __restrict__ hout,
                                                  double* __restrict__ w, int64_t len, double* __restrict__ part_out) {
    __shared__ double h[kFuseCols], sh[4];
    reduce_columns(part_in, k, h);
    if (blockIdx.x == 0 && (int)threadIdx.x < k) hout[threadIdx.x] = h[threadIdx.x];
    double q = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (int64_t)kRedBlocks * 256) {
        double s = 0.0;
#pragma unroll 4
        for (int j = 0; j < k; ++j) s = fma(h[j], V[(int64_t)j * ld + i], s);
        const double wi = w[i] - s;
        w[i] = wi;
        q = fma(wi, wi, q);
    }
    const double r = block_sum(q, sh);
    if (threadIdx.x == 0) part_out[blockIdx.x] = r;
    clear_partials(part_out);
}

// out = w / ||w|| (nothing when w = 0); the squared norm to hout
__global__ __launch_bounds__(256) void k_cgs_scale(const double* __restrict__ part_in, double* __restrict__ hout,
                                                   const double* __restrict__ w, double* __restrict__ out, int64_t len) {
    __shared__ double sh;
    if (threadIdx.x < 64) {
        const double r = reduce_blocks(part_in);
        if (threadIdx.x == 0) {
            sh = r;
            if (blockIdx.x == 0) hout[0] = r;
        }
    }
    __syncthreads();
    if (!(sh > 0.0)) return;
    const double a = 1.0 / sqrt(sh);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (int64_t)gridDim.x * 256) out[i] = a * w[i];
}

__global__ void k_multi_axpy(const double* __restrict__ V, int64_t ld, int k, const double* __restrict__ h,
                             double sign, double* __restrict__ w, int64_t len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= len) return;
    double s = 0.0;
    for (int j = 0; j < k; ++j) s += h[j] * V[(int64_t)j * ld + i];
    w[i] += sign * s;
}

// out may alias x or y (elementwise: each lane reads its element before writing it)
__global__ void k_axpby(double a, const double* x, double b, const double* y, double* out, int64_t len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= len) return;
    out[i] = a * x[i] + (y ? b * y[i] : 0.0);
}

__global__ void k_fill(double v, double* __restrict__ out, int64_t len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < len) out[i] = v;
}

__global__ void k_add_scalar(double* __restrict__ x, const double* __restrict__ d, double scale, int64_t len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < len) x[i] += scale * d[0];
}

__global__ void k_normal_comp(int64_t n, const double* __restrict__ nrm, const double* __restrict__ u,
                              double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = nrm[i] * u[i] + nrm[n + i] * u[n + i] + nrm[2 * n + i] * u[2 * n + i];
}

__global__ void k_traction(int64_t n, const double* __restrict__ nrm, const double* __restrict__ p,
                           const double* __restrict__ u, double beta, const double* __restrict__ fx,
                           double* __restrict__ f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double nx = nrm[i], ny = nrm[n + i], nz = nrm[2 * n + i];
    const double pi = p ? p[i] : 0.0;
    double tx = 0.0, ty = 0.0, tz = 0.0;
    if (u && beta != 0.0) {
        const double ux = u[i], uy = u[n + i], uz = u[2 * n + i];
        const double un = ux * nx + uy * ny + uz * nz;
        tx = beta * (ux - un * nx);
        ty = beta * (uy - un * ny);
        tz = beta * (uz - un * nz);
    }
    f[i] = -pi * nx + tx + (fx ? fx[i] : 0.0);
    f[n + i] = -pi * ny + ty + (fx ? fx[n + i] : 0.0);
    f[2 * n + i] = -pi * nz + tz + (fx ? fx[2 * n + i] : 0.0);
}

__global__ void k_gather(int64_t n, int comps, const int32_t* __restrict__ perm, const double* __restrict__ src,
                         double* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = perm[i];
    for (int c = 0; c < comps; ++c) dst[c * n + i] = src[c * n + o];
}

__global__ void k_scatter(int64_t n, int comps, const int32_t* __restrict__ perm, const double* __restrict__ src,
                          double* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = perm[i];
    for (int c = 0; c < comps; ++c) dst[c * n + o] = src[c * n + i];
}

// ---- adjoint helpers ------------------------------------------------------
// out = tn + lam * dl1 + w * (*sum) / area      (transposed completed Darcy operator)
__global__ void k_adj_darcy(int64_t n, const double* __restrict__ tn, const double* __restrict__ lam,
                            const double* __restrict__ dl1, const double* __restrict__ w,
                            const double* __restrict__ sum, double inv_area, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = tn[i] + lam[i] * dl1[i] + w[i] * sum[0] * inv_area;
}

// out = lam + sum_c mneg_c lam_c + tns + w n (*flux)/area + beta P_tau sv, where sv
// already carries the target weight w
// (transposed completed Stokes operator with slip); mneg_c[a][i] = -(M_i)_{ac}
__global__ void k_adj_stokes(int64_t n, const double* __restrict__ lam, const double* __restrict__ m0,
                             const double* __restrict__ m1, const double* __restrict__ m2,
                             const double* __restrict__ tns, const double* __restrict__ sv,
                             const double* __restrict__ nrm, const double* __restrict__ w,
                             const double* __restrict__ flux, double inv_area, double beta, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double l[3] = {lam[i], lam[n + i], lam[2 * n + i]};
    const double nv[3] = {nrm[i], nrm[n + i], nrm[2 * n + i]};
    double svn = 0.0;
    if (sv) svn = sv[i] * nv[0] + sv[n + i] * nv[1] + sv[2 * n + i] * nv[2];
    const double fl = flux[0] * inv_area;
    for (int a = 0; a < 3; ++a) {
        const int64_t k = a * n + i;
        double v = l[a] + m0[k] * l[0] + m1[k] * l[1] + m2[k] * l[2] + tns[k] + w[i] * nv[a] * fl;
        if (sv) v += beta * (sv[k] - svn * nv[a]);  // sv carries the target weight
        out[k] = v;
    }
}

// out3 = scale * s n
__global__ void k_scalar_normal(int64_t n, const double* __restrict__ s, double scale, const double* __restrict__ nrm,
                                double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    for (int c = 0; c < 3; ++c) out[c * n + i] = scale * s[i] * nrm[c * n + i];
}

// x += scale * (*d) * w
__global__ void k_axpy_w(int64_t n, double* __restrict__ x, const double* __restrict__ w, const double* __restrict__ d,
                         double scale) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] += scale * d[0] * w[i];
}

// gp = -w (e.n);  gu = beta w (e - (e.n) n)
__global__ void k_adj_rhs(int64_t n, const double* __restrict__ nrm, const double* __restrict__ w, double e0, double e1,
                          double e2, double beta, double* __restrict__ gp, double* __restrict__ gu) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double nx = nrm[i], ny = nrm[n + i], nz = nrm[2 * n + i];
    const double en = e0 * nx + e1 * ny + e2 * nz;
    gp[i] = -w[i] * en;
    gu[i] = beta * w[i] * (e0 - en * nx);
    gu[n + i] = beta * w[i] * (e1 - en * ny);
    gu[2 * n + i] = beta * w[i] * (e2 - en * nz);
}

inline unsigned nblk(int64_t len) { return (unsigned)((len + 255) / 256); }

}  // namespace

void dev_dot(const Plan& P, const double* a, const double* b, int64_t len, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_dot_partial, dim3(red_blocks(len)), dim3(256), 0, s, a, b, len, P.red);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_reduce_cols, dim3(1), dim3(256), 0, s, (const double*)P.red, kRedBlocks, out);
    SDBIE_LAUNCHED();
}

void dev_multidot(const Plan& P, const double* V, int64_t ld, int k, const double* w, int64_t len,
                  double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_multidot_partial, dim3(kRedBlocks, (unsigned)((k + kDotCols - 1) / kDotCols)), dim3(256), 0,
                       s, V, ld, k, w, len, P.red);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_reduce_cols, dim3(k), dim3(256), 0, s, (const double*)P.red, kRedBlocks, out);
    SDBIE_LAUNCHED();
}

void dev_cgs2(const Plan& P, const double* Vr, int kr, const double* rot, const double* V, int k, double* w,
              double* next, int64_t len, hipStream_t s) {
    double* host = P.host_pinned;
    double* pa = P.red;           // two sets of block partials in turn
    double* pb = P.partial;       // free between the pair passes
    static_assert((size_t)(kFuseCols + 1) * kRedBlocks * sizeof(double) <= (size_t)1 << 20, "block partials in `partial`");
    const bool small = len <= (int64_t)kRedBlocks * 64;
    const dim3 grid(small ? kRedBlocks / 4 : kRedBlocks), th(256);
    const int k0 = kr > 0 ? kr + 1 : k;
    const dim3 g0(grid.x, (unsigned)((k0 + kDotCols - 1) / kDotCols));
    if (small)
        hipLaunchKernelGGL(k_multidot_small, g0, th, 0, s, kr > 0 ? Vr : V, len, k0, (const double*)w, len, pa);
    else
        hipLaunchKernelGGL(k_multidot_partial, g0, th, 0, s, kr > 0 ? Vr : V, len, k0, (const double*)w, len, pa);
    SDBIE_LAUNCHED();
    auto step = [&](const double* Vs, int ks, const double* r, double* h) {
        if (small)
            hipLaunchKernelGGL((k_cgs_step<true>), grid, th, 0, s, Vs, len, ks, (const double*)pa, r, h, V, len, k, w,
                               len, pb);
        else
            hipLaunchKernelGGL((k_cgs_step<false>), grid, th, 0, s, Vs, len, ks, (const double*)pa, r, h, V, len, k, w,
                               len, pb);
        SDBIE_LAUNCHED();
        std::swap(pa, pb);
    };
    if (kr > 0) step(Vr, kr + 1, rot, host + kHostE);
    step(V, k, nullptr, host + kHostH1);
    hipLaunchKernelGGL(k_cgs_last, dim3(red_blocks(len)), th, 0, s, V, len, k, (const double*)pa, host + kHostH2, w, len,
                       pb);
    SDBIE_LAUNCHED();
    const unsigned sb = nblk(len) < kRedBlocks ? nblk(len) : kRedBlocks;
    hipLaunchKernelGGL(k_cgs_scale, dim3(sb), th, 0, s, (const double*)pb, host + kHostNorm, (const double*)w, next, len);
    SDBIE_LAUNCHED();
}

double dev_dot_host(const Plan& P, const double* a, const double* b, int64_t len, hipStream_t s) {
    double* part = P.host_pinned + kHostDot;
    hipLaunchKernelGGL(k_dot_partial, dim3(red_blocks(len)), dim3(256), 0, s, a, b, len, part);
    SDBIE_LAUNCHED();
    SDBIE_HIP(hipStreamSynchronize(s));
    // k_reduce_cols' order
    double r[4];
    for (int v = 0; v < 4; ++v) {
        double t[64];
        for (int l = 0; l < 64; ++l) t[l] = part[64 * v + l] + part[64 * v + l + 256];
        for (int o = 32; o > 0; o >>= 1)
            for (int l = 0; l < o; ++l) t[l] += t[l + o];
        r[v] = t[0];
    }
    return (r[0] + r[1]) + (r[2] + r[3]);
}

void dev_multi_axpy_sub(const double* V, int64_t ld, int k, const double* h, double* w, int64_t len,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_multi_axpy, dim3(nblk(len)), dim3(256), 0, s, V, ld, k, h, -1.0, w, len);
    SDBIE_LAUNCHED();
}

void dev_multi_axpy_add(const double* V, int64_t ld, int k, const double* y, double* x, int64_t len,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_multi_axpy, dim3(nblk(len)), dim3(256), 0, s, V, ld, k, y, 1.0, x, len);
    SDBIE_LAUNCHED();
}

void dev_axpby(double a, const double* x, double b, const double* y, double* out, int64_t len, hipStream_t s) {
    hipLaunchKernelGGL(k_axpby, dim3(nblk(len)), dim3(256), 0, s, a, x, b, y, out, len);
    SDBIE_LAUNCHED();
}

void dev_scale(double a, const double* x, double* out, int64_t len, hipStream_t s) {
    dev_axpby(a, x, 0.0, nullptr, out, len, s);
}

void dev_fill(double v, double* out, int64_t len, hipStream_t s) {
    hipLaunchKernelGGL(k_fill, dim3(nblk(len)), dim3(256), 0, s, v, out, len);
    SDBIE_LAUNCHED();
}

void dev_add_scaled_scalar(double* x, const double* d, double scale, int64_t len, hipStream_t s) {
    hipLaunchKernelGGL(k_add_scalar, dim3(nblk(len)), dim3(256), 0, s, x, d, scale, len);
    SDBIE_LAUNCHED();
}

void dev_normal_component(const Plan& P, const double* u, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_normal_comp, dim3(nblk(P.n)), dim3(256), 0, s, P.n, (const double*)P.nrm, u, out);
    SDBIE_LAUNCHED();
}

void dev_traction(const Plan& P, const double* p, const double* u, double beta, const double* f_extra,
                  double* f, hipStream_t s) {
    hipLaunchKernelGGL(k_traction, dim3(nblk(P.n)), dim3(256), 0, s, P.n, (const double*)P.nrm, p, u, beta,
                       f_extra, f);
    SDBIE_LAUNCHED();
}

void dev_gather(const Plan& P, const double* src, double* dst, int comps, hipStream_t s) {
    hipLaunchKernelGGL(k_gather, dim3(nblk(P.n)), dim3(256), 0, s, P.n, comps, (const int32_t*)P.perm, src, dst);
    SDBIE_LAUNCHED();
}

void dev_scatter(const Plan& P, const double* src, double* dst, int comps, hipStream_t s) {
    hipLaunchKernelGGL(k_scatter, dim3(nblk(P.n)), dim3(256), 0, s, P.n, comps, (const int32_t*)P.perm, src, dst);
    SDBIE_LAUNCHED();
}

void dev_adj_darcy(const Plan& P, const double* tn, const double* lam, const double* dl1, const double* sum,
                   double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_darcy, dim3(nblk(P.n)), dim3(256), 0, s, P.n, tn, lam, dl1, (const double*)P.w, sum,
                       1.0 / P.area, out);
    SDBIE_LAUNCHED();
}

void dev_adj_stokes(const Plan& P, const double* lam, const double* m0, const double* m1, const double* m2,
                    const double* tns, const double* sv, const double* flux, double beta, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_stokes, dim3(nblk(P.n)), dim3(256), 0, s, P.n, lam, m0, m1, m2, tns, sv,
                       (const double*)P.nrm, (const double*)P.w, flux, 1.0 / P.area, beta, out);
    SDBIE_LAUNCHED();
}

void dev_scalar_normal(const Plan& P, const double* sv, double scale, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_scalar_normal, dim3(nblk(P.n)), dim3(256), 0, s, P.n, sv, scale, (const double*)P.nrm, out);
    SDBIE_LAUNCHED();
}

void dev_axpy_w(const Plan& P, double* x, const double* d, double scale, hipStream_t s) {
    hipLaunchKernelGGL(k_axpy_w, dim3(nblk(P.n)), dim3(256), 0, s, P.n, x, (const double*)P.w, d, scale);
    SDBIE_LAUNCHED();
}

void dev_adj_rhs(const Plan& P, const double e[3], double beta, double* gp, double* gu, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_rhs, dim3(nblk(P.n)), dim3(256), 0, s, P.n, (const double*)P.nrm, (const double*)P.w, e[0],
                       e[1], e[2], beta, gp, gu);
    SDBIE_LAUNCHED();
}

}  // namespace sdbie
