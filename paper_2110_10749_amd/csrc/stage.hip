// Surface staging: spatial (Morton) order and the sorted node copies.
//
// The pair kernels give each wave 64 consecutive targets; sorting the nodes
// along a Morton (Z-order) curve makes those 64 targets spatial neighbours,
// so the near-field branch (rho < rho_cut) is taken by few waves per source
// and the rest run the plain far-field kernel.
//
// Steps (all on the device, one synchronisation at the end): finite check and
// bounding box; 30-bit Morton key per node (10 bits per axis), key<<32 | index
// sorted by a bitonic network over the next power of two (padding keys =
// UINT64_MAX; keys are unique, so the order is deterministic); gather of x, n,
// w into sorted double arrays and the weighted normals w n, copies padded to
// whole tiles of kTile nodes for the pair kernels, tile and unit bounding
// boxes and a float copy of the coordinates in the frame of each node's tile;
// the near-field masks of tile pairs (box distance below rho_cut delta, one
// mask for the double cutoff and one for the float cutoff); and the work lists
// of the symmetric passes.
//
// Staging is launches more than work: with one launch per step of the sorting
// network (153 at n = 68166), one per array and three synchronisations it took
// 0.8 ms there and 0.45 ms at n = 9582; now about 20 launches and 0.2 ms.
#include "smoothing_coeffs.h"
#include "solver.h"

namespace sdbie {
namespace {

constexpr int kScanBlocks = 256;  // blocks of the input scan

// per block: min and max of x per axis, then 1 if some entry of x, n or w is
// not finite, 1 if some coordinate exceeds kMaxCoord: part[kScanBlocks][8]
__global__ __launch_bounds__(256) void k_scan_input(int64_t n, const double* __restrict__ x,
                                                    const double* __restrict__ nrm, const double* __restrict__ w,
                                                    double* __restrict__ part) {
    __shared__ double sh[4][8];
    double v[8] = {INFINITY, -INFINITY, INFINITY, -INFINITY, INFINITY, -INFINITY, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)kScanBlocks * 256) {
        for (int c = 0; c < 3; ++c) {
            const double t = x[c * n + i];
            v[2 * c] = fmin(v[2 * c], t);
            v[2 * c + 1] = fmax(v[2 * c + 1], t);
            if (!isfinite(t) || !isfinite(nrm[c * n + i])) v[6] = 1.0;
            else if (fabs(t) > kMaxCoord) v[7] = 1.0;
        }
        if (!isfinite(w[i])) v[6] = 1.0;
    }
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double t = __shfl_xor(v[c], o, 64);
            v[c] = c < 6 && !(c & 1) ? fmin(v[c], t) : fmax(v[c], t);
        }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 8; ++c) sh[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x < 8) {
        const int c = threadIdx.x;
        double r = sh[0][c];
        for (int k = 1; k < 4; ++k) r = c < 6 && !(c & 1) ? fmin(r, sh[k][c]) : fmax(r, sh[k][c]);
        part[blockIdx.x * 8 + c] = r;
    }
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Morton keys; every block adds up the block results of the input scan, the
// first writes them to stage[0..9] (the box 2 .. 7, the two flags as ints in
// stage[0]) and clears the near-pair counters stage[10], stage[11]
__global__ __launch_bounds__(256) void k_morton(int64_t n, int64_t npow2, const double* __restrict__ x,
                                                const double* __restrict__ part, double* __restrict__ stage,
                                                uint64_t* __restrict__ keys) {
    __shared__ double sh[4][8], bb[8];
    static_assert(kScanBlocks == 256, "one block result per thread");
    double v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = part[threadIdx.x * 8 + c];
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double t = __shfl_xor(v[c], o, 64);
            v[c] = c < 6 && !(c & 1) ? fmin(v[c], t) : fmax(v[c], t);
        }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 8; ++c) sh[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x < 8) {
        const int c = threadIdx.x;
        double r = sh[0][c];
        for (int k = 1; k < 4; ++k) r = c < 6 && !(c & 1) ? fmin(r, sh[k][c]) : fmax(r, sh[k][c]);
        bb[c] = r;
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        int* flag = reinterpret_cast<int*>(stage);
        flag[0] = bb[6] > 0.0;
        flag[1] = bb[7] > 0.0;
        for (int c = 0; c < 6; ++c) stage[2 + c] = bb[c];
        stage[10] = stage[11] = 0.0;  // two 64-bit counters (all-zero bits)
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= npow2) return;
    if (i >= n) {
        keys[i] = ~0ull;
        return;
    }
    uint32_t code = 0;
    // a cube of the largest extent, so the curve is isotropic
    const double ext = fmax(fmax(bb[1] - bb[0], bb[3] - bb[2]), bb[5] - bb[4]);
    const double sc = ext > 0.0 ? 1023.0 / ext : 0.0;
    for (int c = 0; c < 3; ++c) {
        double t = (x[c * n + i] - bb[2 * c]) * sc;
        t = fmin(fmax(t, 0.0), 1023.0);
        code |= spread10((uint32_t)t) << (2 - c);
    }
    keys[i] = ((uint64_t)code << 32) | (uint64_t)i;
}

// ---- sorting network -----------------------------------------------------------
// Bitonic steps (k, j) compare elements i and i ^ j; the lower one keeps the
// smaller key where bit k of i is clear.  A block holds kSortBlock consecutive
// keys, 8 to a thread (with 8192 the passes of one block, bound by the LDS pipe,
// took 21 to 32 us each: 132 us of sorting at n = 68166): steps with j < 8 stay in registers, j < 512 pass keys
// between the lanes of a wave, the others through LDS.  Steps across blocks run
// up to three to a launch, 8 keys to a thread.
constexpr int kSortBlock = 2048, kSortThreads = kSortBlock / 8;

__device__ __forceinline__ uint64_t keep(uint64_t a, uint64_t b, bool smaller) {
    return (a < b) == smaller ? a : b;
}

// steps k, j = jmax, jmax / 2 .. 1 on the block's keys (element i0 + 8 tid + e in v[e])
__device__ __forceinline__ void bitonic_block(uint64_t (&v)[8], int64_t i0, int64_t k, int jmax, uint64_t* sh) {
    const int tid = threadIdx.x;
    const int64_t i = i0 + 8 * tid;
    for (int j = jmax; j >= 8; j >>= 1) {
        const bool smaller = ((i & k) == 0) == ((i & j) == 0);  // bits above the 8 elements of a thread
        if (j >= 512) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 8; ++e) sh[e * kSortThreads + tid] = v[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = keep(v[e], sh[e * kSortThreads + (tid ^ (j >> 3))], smaller);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = keep(v[e], (uint64_t)__shfl_xor((unsigned long long)v[e], j >> 3, 64), smaller);
        }
    }
#pragma unroll
    for (int j = 4; j > 0; j >>= 1) {
        if (j > jmax) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (!(e & j)) {
                const bool up = ((i + e) & k) == 0;
                const uint64_t a = v[e], b = v[e | j];
                v[e] = keep(a, b, up);
                v[e | j] = keep(a, b, !up);
            }
    }
}

// full: every step k = 2 .. min(npow2, kSortBlock); else the steps j < kSortBlock of k
__global__ __launch_bounds__(kSortThreads) void k_sort_block(uint64_t* __restrict__ keys, int64_t npow2, int64_t k,
                                                             int full) {
    __shared__ uint64_t sh[kSortBlock];
    const int64_t i0 = (int64_t)blockIdx.x * kSortBlock, i = i0 + 8 * threadIdx.x;
    uint64_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = i + e < npow2 ? keys[i + e] : ~0ull;
    if (full) {
        const int64_t top = npow2 < kSortBlock ? npow2 : kSortBlock;
        for (int64_t kk = 2; kk <= top; kk <<= 1) bitonic_block(v, i0, kk, (int)(kk >> 1), sh);
    } else {
        bitonic_block(v, i0, k, kSortBlock / 2, sh);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (i + e < npow2) keys[i + e] = v[e];
}

// steps (k, j), (k, j / 2) .. (k, j >> (S - 1)) across blocks: 2^S keys to a thread, j >> (S - 1) apart
template <int S>
__global__ __launch_bounds__(256) void k_sort_global(uint64_t* __restrict__ keys, int64_t npow2, int64_t k, int64_t j) {
    constexpr int E = 1 << S;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, d = j >> (S - 1);
    if (t >= npow2 / E) return;
    const int64_t i = (t / d) * (d * E) + t % d;  // the S bits from log2 d on are clear
    const bool up = (i & k) == 0;                 // k > j: the same for the thread's keys
    uint64_t v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = keys[i + e * d];
#pragma unroll
    for (int b = E / 2; b > 0; b >>= 1)
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (!(e & b)) {
                const uint64_t x = v[e], y = v[e | b];
                v[e] = keep(x, y, up);
                v[e | b] = keep(x, y, !up);
            }
#pragma unroll
    for (int e = 0; e < E; ++e) keys[i + e * d] = v[e];
}

void sort_keys(uint64_t* keys, int64_t npow2, hipStream_t st) {
    const unsigned nb = (unsigned)((npow2 + kSortBlock - 1) / kSortBlock);
    // one wave at least; below kSortBlock only the threads that hold keys
    const unsigned th = npow2 >= kSortBlock ? kSortThreads : (unsigned)(npow2 / 8 < 64 ? 64 : npow2 / 8);
    hipLaunchKernelGGL(k_sort_block, dim3(nb), dim3(th), 0, st, keys, npow2, (int64_t)0, 1);
    SDBIE_LAUNCHED();
    for (int64_t k = 2 * kSortBlock; k <= npow2; k <<= 1) {
        int64_t j = k >> 1;
        while (j >= kSortBlock) {
            const int64_t left = j / kSortBlock;  // steps left across blocks: log2(left) + 1
            const int s = left >= 4 ? 3 : left >= 2 ? 2 : 1;
            const dim3 g((unsigned)(((npow2 >> s) + 255) / 256));
            if (s == 3) hipLaunchKernelGGL((k_sort_global<3>), g, dim3(256), 0, st, keys, npow2, k, j);
            else if (s == 2) hipLaunchKernelGGL((k_sort_global<2>), g, dim3(256), 0, st, keys, npow2, k, j);
            else hipLaunchKernelGGL((k_sort_global<1>), g, dim3(256), 0, st, keys, npow2, k, j);
            SDBIE_LAUNCHED();
            j >>= s;
        }
        hipLaunchKernelGGL(k_sort_block, dim3(nb), dim3(kSortThreads), 0, st, keys, npow2, k, 0);
        SDBIE_LAUNCHED();
    }
}

// Sorted and padded copies, one block per tile.  Padding nodes k >= n sit at a
// point outside the bounding box (10 extents away) with zero weight and normal.
// Boxes of the tile and of its units hold the real nodes (empty: +inf / -inf).
// The float coordinates are in the frame of their tile: minus the centre of the
// tile's box (every tile holds at least one real node, so the centre is finite).
// The kernels see coordinates only through differences x_i - x_j, formed after
// moving the targets into the source tile's frame, so the rounding of a float
// coordinate is set by the tile's extent, not by the body's or by the
// distance from the origin.
struct StageArgs {
    int64_t n, npad;
    const uint64_t* keys;
    const double *x, *nrm, *w, *bb;  // bb: bounding box
    int32_t* perm;
    double *xs, *ns, *ws, *wn, *px, *pn, *pw;
    float* px32;
    double *boxes, *uboxes;
};

__global__ __launch_bounds__(kTile) void k_stage(StageArgs a) {
    __shared__ double ub[kTile / 64][6];
    static_assert(kNearUnit == 64, "a wave stages a unit");
    const int64_t k = (int64_t)blockIdx.x * kTile + threadIdx.x, n = a.n, npad = a.npad;
    const bool real = k < n;
    const int64_t o = real ? (int64_t)(a.keys[k] & 0xffffffffull) : 0;
    const double ext = fmax(fmax(a.bb[1] - a.bb[0], a.bb[3] - a.bb[2]), a.bb[5] - a.bb[4]);
    const double wk = real ? a.w[o] : 0.0;
    double xv[3], lo[3], hi[3];
    for (int c = 0; c < 3; ++c) {
        xv[c] = real ? a.x[c * n + o] : a.bb[2 * c + 1] + 10.0 * ext + 1.0;
        const double nv = real ? a.nrm[c * n + o] : 0.0;
        if (real) {
            a.xs[c * n + k] = xv[c];
            a.ns[c * n + k] = nv;
            a.wn[c * n + k] = wk * nv;
        }
        a.px[c * npad + k] = xv[c];
        a.pn[c * npad + k] = nv;
        lo[c] = real ? xv[c] : INFINITY;
        hi[c] = real ? xv[c] : -INFINITY;
    }
    if (real) {
        a.perm[k] = (int32_t)o;
        a.ws[k] = wk;
    }
    a.pw[k] = wk;
    for (int off = 32; off > 0; off >>= 1)
        for (int c = 0; c < 3; ++c) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], off, 64));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], off, 64));
        }
    const int u = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < 3; ++c) {
            ub[u][2 * c] = lo[c];
            ub[u][2 * c + 1] = hi[c];
        }
    __syncthreads();
    for (int c = 0; c < 3; ++c) {
        lo[c] = fmin(fmin(ub[0][2 * c], ub[1][2 * c]), fmin(ub[2][2 * c], ub[3][2 * c]));
        hi[c] = fmax(fmax(ub[0][2 * c + 1], ub[1][2 * c + 1]), fmax(ub[2][2 * c + 1], ub[3][2 * c + 1]));
        a.px32[c * npad + k] = (float)(xv[c] - 0.5 * (lo[c] + hi[c]));
    }
    if (threadIdx.x < 6) {
        const int c = threadIdx.x;
        double r = ub[0][c];
        for (int k = 1; k < 4; ++k) r = c & 1 ? fmax(r, ub[k][c]) : fmin(r, ub[k][c]);
        a.boxes[(int64_t)blockIdx.x * 6 + c] = r;
    }
    if (threadIdx.x < 24) a.uboxes[(int64_t)blockIdx.x * 24 + threadIdx.x] = ub[threadIdx.x / 6][threadIdx.x % 6];
}

// Near masks, and the work lists of the symmetric passes, in three kernels: the
// mask rows and their counts, the prefix sums of those (one block), and the
// items and blocks of each row.  Blocks hold as many pairs as leave about
// SDBIE_SYM_TARGET of them for each kind of pair (at most kSymChunk while the
// forward slots have room).  More pairs to a block save target loads and forward
// slots, fewer let the last wave of blocks end together: with targets of 2048 and
// 16384 (4096, 8192 and 65536 lie between or are equal) n = 68166 takes, us a pass,
// 3895 and 3760 for the double Stokes double layer, 2720 and 2605 for the float
// slip sum, 1333 and 1255 for the float Laplace double layer.

// position of this thread's flag among the set flags of the block (256 threads), and their number
__device__ __forceinline__ int block_rank(bool f, int* sh, int& total) {
    const uint64_t bal = __ballot(f);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = __popcll(bal);
    __syncthreads();
    int before = __popcll(bal & ((1ull << lane) - 1));
    total = 0;
    for (int k = 0; k < 4; ++k) {
        if (k < w) before += sh[k];
        total += sh[k];
    }
    __syncthreads();
    return before;
}

// ints of a row in sym_rows: counts, then (k_list_scan) starts
enum : int {
    kRowNear64 = 0,  // near pairs b > a (double)
    kRowFar64,       // far pairs b > a
    kRowColFar64,    // far pairs b < a
    kRowNear32,      // near pairs b != a (float)
    kRowFar32,       // far pairs b > a
    kRowItem,        // first item: double, float, far-only (3)
    kRowNearBlk = kRowItem + 3,    // first near block: double, float (2)
    kRowFarBlk = kRowNearBlk + 2,  // first far block: double, float, far-only (3)
};
static_assert(kRowFarBlk + 3 <= kSymRowInts, "ints of a row");

// mask[a][b] = 1 when the boxes of tiles a and b are closer than the cutoff (one
// block per row a; the masks are symmetric).  cnt[0], cnt[1] += the (target,
// source) pairs of real nodes in the near tile pairs of each precision (integer
// sums: exact in any order).  With rows: the counts of the row's tile pairs, and
// for the far-only set the rank of each far b < a in column a.  The first
// kRedBlocks blocks also take the block partials of the weight sum (dev_dot's).
__global__ __launch_bounds__(256) void k_mask_rows(int T, int64_t n, const double* __restrict__ boxes, double rc64,
                                                   double rc32, uint8_t* __restrict__ m64, uint8_t* __restrict__ m32,
                                                   unsigned long long* __restrict__ cnt, int32_t* __restrict__ rows,
                                                   int32_t* __restrict__ colrank, const double* __restrict__ w,
                                                   double* __restrict__ part) {
    __shared__ int sh[4];
    __shared__ double shd[4];
    const int a = blockIdx.x;
    if (a < kRedBlocks) {
        double s = 0.0;
        for (int64_t i = (int64_t)a * 256 + threadIdx.x; i < n; i += (int64_t)kRedBlocks * 256) s += w[i];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if ((threadIdx.x & 63) == 0) shd[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) part[a] = (shd[0] + shd[1]) + (shd[2] + shd[3]);
    }
    if (a >= T) return;
    // wave v takes the 64-tile groups g = v, v + 4, ..; the counts stay in its scalars
    __shared__ int cnt5[4][5], before[kSymMaxTiles / 64 + 1];
    const double* A = boxes + (int64_t)a * 6;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, groups = (T + 63) / 64;
    int c[5] = {0, 0, 0, 0, 0};
    unsigned long long c64 = 0, c32 = 0;
    for (int g = wave; g < groups; g += 4) {
        const int b = 64 * g + lane;
        const bool in = b < T;
        bool n64 = false, n32 = false;
        if (in) {
            const double* B = boxes + (int64_t)b * 6;
            double d2 = 0.0;
            for (int k = 0; k < 3; ++k) {
                const double gap = fmax(0.0, fmax(A[2 * k] - B[2 * k + 1], B[2 * k] - A[2 * k + 1]));
                d2 += gap * gap;
            }
            n64 = d2 < rc64 * rc64;
            n32 = d2 < rc32 * rc32;
            m64[(int64_t)a * T + b] = n64 ? 1 : 0;
            m32[(int64_t)a * T + b] = n32 ? 1 : 0;
            const int64_t ra = n - (int64_t)a * kTile < kTile ? n - (int64_t)a * kTile : kTile;
            const int64_t rb = n - (int64_t)b * kTile < kTile ? n - (int64_t)b * kTile : kTile;
            if (n64) c64 += (unsigned long long)(ra * rb);
            if (n32) c32 += (unsigned long long)(ra * rb);
        }
        if (!rows) continue;
        const uint64_t cf = __ballot(in && b < a && !n64);
        c[kRowNear64] += __popcll(__ballot(in && b > a && n64));
        c[kRowFar64] += __popcll(__ballot(in && b > a && !n64));
        c[kRowColFar64] += __popcll(cf);
        c[kRowNear32] += __popcll(__ballot(in && b != a && n32));
        c[kRowFar32] += __popcll(__ballot(in && b > a && !n32));
        if (lane == 0) before[g + 1] = __popcll(cf);
    }
    if (rows) {
        if (lane == 0)
            for (int k = 0; k < 5; ++k) cnt5[wave][k] = c[k];
        __syncthreads();
        if (threadIdx.x < 5)
            rows[(int64_t)a * kSymRowInts + threadIdx.x] =
                cnt5[0][threadIdx.x] + cnt5[1][threadIdx.x] + cnt5[2][threadIdx.x] + cnt5[3][threadIdx.x];
        if (threadIdx.x == 0) {
            before[0] = 0;
            for (int g = 0; g < groups; ++g) before[g + 1] += before[g];
        }
        __syncthreads();
        for (int g = wave; g < groups && 64 * g < a; g += 4) {
            const int b = 64 * g + lane;
            const bool f = b < a && !m64[(int64_t)a * T + (b < T ? b : 0)];  // this wave's own writes
            const uint64_t cf = __ballot(f);
            if (f) colrank[(int64_t)a * T + b] = before[g] + __popcll(cf & ((1ull << lane) - 1));
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        c64 += __shfl_down(c64, off);
        c32 += __shfl_down(c32, off);
    }
    if ((threadIdx.x & 63) == 0) {
        if (c64) atomicAdd(cnt, c64);
        if (c32) atomicAdd(cnt + 1, c32);
    }
}

// the weight sum from its block partials (k_reduce_cols' order)
__device__ __forceinline__ void reduce_area(const double* __restrict__ part, double* __restrict__ out) {
    __shared__ double sh[4];
    double s = part[threadIdx.x] + part[threadIdx.x + 256];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}
__global__ __launch_bounds__(256) void k_area(const double* __restrict__ part, double* __restrict__ out) {
    reduce_area(part, out);
}

struct ListArgs {
    int T;
    int parts[2], self_parts[2];  // double, float
    int room[2];                  // forward slots
    const uint8_t* mask[2];
    const int32_t* colrank;
    int32_t* rows;
    int32_t *items[3], *blocks[3], *fwd_start[3], *rev_start[3];
    int32_t* out;  // number of blocks of the three sets, near and far chunk of double and float
    const double* area_part;
    double* area;
};

constexpr int kScanRows = kSymMaxTiles / 256;  // rows per thread of the scan

// exclusive prefix sums over the rows of v[0..kScanRows) (thread-consecutive), total over all
__device__ __forceinline__ int block_scan(int (&v)[kScanRows], int* sh) {
    int s = 0;
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
        const int t = v[i];
        v[i] = s;
        s += t;
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = s;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int base = inc - s, total = 0;
    for (int k = 0; k < 4; ++k) {
        if (k < w) base += sh[k];
        total += sh[k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] += base;
    return total;
}

__global__ __launch_bounds__(256) void k_list_scan(ListArgs A) {
    __shared__ int sh[4];
    reduce_area(A.area_part, A.area);
    const int r0 = threadIdx.x * kScanRows;
    auto row = [&](int i, int what) { return r0 + i < A.T ? A.rows[(int64_t)(r0 + i) * kSymRowInts + what] : 0; };
    auto put = [&](int i, int what, int v) {
        if (r0 + i < A.T) A.rows[(int64_t)(r0 + i) * kSymRowInts + what] = v;
    };
    int v[kScanRows];
    for (int k = 0; k < 2; ++k) {
        const int wn = k ? kRowNear32 : kRowNear64, wf = k ? kRowFar32 : kRowFar64, parts = A.parts[k];
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) v[i] = r0 + i < A.T ? 1 + row(i, wn) : 0;
        const int near = block_scan(v, sh);
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) v[i] = row(i, wf);
        const int far = block_scan(v, sh);
        int nc = min(max(near / SDBIE_SYM_TARGET, 1), kSymChunk), fc = min(max(far / SDBIE_SYM_TARGET, 1), kSymChunk);
        if (parts > 1) nc = fc = 1;
        else
            while (near / nc + far / fc + 2 * A.T > A.room[k]) {  // room holds 2 T slots and more
                ++nc;
                ++fc;
            }
        auto near_items = [&](int i) { return A.self_parts[k] + row(i, wn) * parts; };
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) v[i] = r0 + i < A.T ? near_items(i) + row(i, wf) * parts : 0;
        block_scan(v, sh);
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) put(i, kRowItem + k, v[i]);
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) v[i] = r0 + i < A.T ? (near_items(i) + nc - 1) / nc : 0;
        const int nb = block_scan(v, sh);
        int fwd[kScanRows];
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) {
            put(i, kRowNearBlk + k, v[i]);
            fwd[i] = v[i];
        }
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) v[i] = (row(i, wf) * parts + fc - 1) / fc;
        const int fb = block_scan(v, sh);
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) {
            put(i, kRowFarBlk + k, nb + v[i]);
            const int b = r0 + i;
            if (b < A.T) {
                A.fwd_start[k][b] = fwd[i] + v[i];
                A.rev_start[k][b] = b * (b - 1) / 2 * parts;
            }
        }
        if (threadIdx.x == 0) {
            A.fwd_start[k][A.T] = nb + fb;
            A.rev_start[k][A.T] = A.T * (A.T - 1) / 2 * parts;
            A.out[k] = nb + fb;
            A.out[3 + 2 * k] = nc;
            A.out[4 + 2 * k] = fc;
        }
    }
    // far pairs alone
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] = row(i, kRowFar64);
    block_scan(v, sh);
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) put(i, kRowItem + 2, v[i]);
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] = (row(i, kRowFar64) + kSymChunk - 1) / kSymChunk;
    const int fb = block_scan(v, sh);
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
        put(i, kRowFarBlk + 2, v[i]);
        if (r0 + i < A.T) A.fwd_start[2][r0 + i] = v[i];
    }
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] = row(i, kRowColFar64);
    const int np = block_scan(v, sh);
#pragma unroll
    for (int i = 0; i < kScanRows; ++i)
        if (r0 + i < A.T) A.rev_start[2][r0 + i] = v[i];
    if (threadIdx.x == 0) {
        A.fwd_start[2][A.T] = fb;
        A.rev_start[2][A.T] = np;
        A.out[2] = fb;
    }
}

__global__ __launch_bounds__(256) void k_list_fill(ListArgs A) {
    __shared__ int sh[4];
    const int a = blockIdx.x, T = A.T;
    const int32_t* row = A.rows + (int64_t)a * kSymRowInts;
    // item `idx` of `total` of one kind (near or far) of this row; `slot0`: the kind's first forward slot
    auto item = [&](int k, int first, int idx, int total, int chunk, int blk0, int slot0, int b, int p, int steps) {
        int32_t* it = A.items[k] + (int64_t)(first + idx) * 4;
        it[0] = a;
        it[1] = b;
        it[2] = p;
        it[3] = steps;
        if (idx % chunk == 0) {
            int32_t* bl = A.blocks[k] + (int64_t)(blk0 + idx / chunk) * 3;
            bl[0] = first + idx;
            bl[1] = total - idx < chunk ? total - idx : chunk;
            bl[2] = slot0 + idx / chunk;
        }
    };
    for (int k = 0; k < 2; ++k) {
        const bool both = k == 1;
        const int parts = A.parts[k], width = 16 / parts, one = (1 << width) - 1;
        const int nc = A.out[3 + 2 * k], fc = A.out[4 + 2 * k];
        const int nnear = A.self_parts[k] + row[both ? kRowNear32 : kRowNear64] * parts;
        const int nfar = row[both ? kRowFar32 : kRowFar64] * parts;
        const int first = row[kRowItem + k], slot = A.fwd_start[k][a], nblk = (nnear + nc - 1) / nc;
        if ((int)threadIdx.x < A.self_parts[k])
            item(k, first, threadIdx.x, nnear, nc, row[kRowNearBlk + k], slot, a, 0,
                 ((one << (threadIdx.x * width)) & (both ? kSymAll : kSymSelf)) | kSymNear);
        int near = 0, far = 0;
        for (int b0 = 0; b0 < T; b0 += 256) {
            const int b = b0 + threadIdx.x;
            const bool m = b < T && A.mask[k][(int64_t)a * T + b];
            int t;
            const bool fn = m && (b > a || (both && b < a));
            const int rn = block_rank(fn, sh, t);
            if (fn)
                for (int q = 0; q < parts; ++q)
                    item(k, first, A.self_parts[k] + (near + rn) * parts + q, nnear, nc, row[kRowNearBlk + k], slot, b,
                         b > a ? (b * (b - 1) / 2 + a) * parts + q : 0, (one << (q * width)) | kSymNear);
            near += t;
            const bool ff = b < T && b > a && !m;
            const int rf = block_rank(ff, sh, t);
            if (ff)
                for (int q = 0; q < parts; ++q)
                    item(k, first + nnear, (far + rf) * parts + q, nfar, fc, row[kRowFarBlk + k], slot + nblk, b,
                         (b * (b - 1) / 2 + a) * parts + q, one << (q * width));
            far += t;
        }
    }
    int far = 0;
    for (int b0 = 0; b0 < T; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const bool f = b < T && b > a && !A.mask[0][(int64_t)a * T + b];
        int t;
        const int r = block_rank(f, sh, t);
        if (f)
            item(2, row[kRowItem + 2], far + r, row[kRowFar64], kSymChunk, row[kRowFarBlk + 2], A.fwd_start[2][a], b,
                 A.rev_start[2][b] + A.colrank[(int64_t)b * T + a], kSymAll);
        far += t;
    }
}

// Enqueues the list kernels after k_mask_rows; the block counts arrive in out[0..2] (device).
// Forward and reverse slots of several parts to a pair share the partial
// buffer of the one-direction passes; of one part the reverse slots have their
// own region, and the forward ones take the larger of the buffer and sym_fwd.
void build_symmetric_lists(Plan& P, int32_t* out, hipStream_t st) {
    const int T = P.ntiles;
    const int64_t pairs = (int64_t)T * (T - 1) / 2;
    ListArgs A;
    A.T = T;
    A.mask[0] = P.mask64;
    A.mask[1] = P.mask32;
    A.rows = P.sym_rows;
    A.colrank = static_cast<const int32_t*>(P.rec);  // T^2 ints; no pass runs yet
    A.out = out;
    A.area_part = P.red;
    A.area = P.scal + kScalStage + 8;
    const bool in_partial = P.partial_bytes > P.sym_fwd_bytes;
    for (int k = 0; k < 2; ++k) {
        SymSet& S = P.sym[k];
        const int64_t items = k == kSymF32 ? (int64_t)T * T : pairs + T;  // at most, of one part
        S.parts = sym_parts(T);
        while (S.parts > 1 && (items + pairs) * S.parts * kSymSlotBytes > P.partial_bytes) S.parts /= 2;
        A.parts[k] = S.parts;
        const int width = 16 / S.parts;
        A.self_parts[k] = k == kSymF32 ? S.parts : (10 + width - 1) / width;  // parts with a step of kSymSelf
        if (S.parts > 1) {
            S.fwd = P.partial;
            S.rev = reinterpret_cast<char*>(P.partial) + (size_t)items * S.parts * kSymSlotBytes;
            A.room[k] = (int)(items * S.parts);
        } else {
            S.fwd = in_partial ? P.partial : static_cast<double*>(P.sym_fwd_mem);
            S.rev = P.sym_rev_mem;
            A.room[k] = (int)((in_partial ? P.partial_bytes : P.sym_fwd_bytes) / kSymSlotBytes);
        }
    }
    P.sym[kSymFar64].fwd = static_cast<double*>(P.sym_fwd_mem);  // the near blocks write to `partial`
    P.sym[kSymFar64].rev = P.sym_rev_mem;
    for (int k = 0; k < 3; ++k) {
        A.items[k] = P.sym[k].items;
        A.blocks[k] = P.sym[k].blocks;
        A.fwd_start[k] = P.sym[k].fwd_start;
        A.rev_start[k] = P.sym[k].rev_start;
    }
    hipLaunchKernelGGL(k_list_scan, dim3(1), dim3(256), 0, st, A);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_list_fill, dim3((unsigned)T), dim3(256), 0, st, A);
    SDBIE_LAUNCHED();
}

}  // namespace

void stage_surface(Plan& P, const sdbie_surface* s, hipStream_t st) {
    const int64_t n = P.n;
    // Flags and counters are written by kernels, not memset nodes (the staging of
    // the allocation-free entry point may sit in a captured stream).  Non-finite
    // input is found at the end: no step reads or writes out of range for it.
    double* stage = P.scal + kScalStage;
    hipLaunchKernelGGL(k_scan_input, dim3(kScanBlocks), dim3(256), 0, st, n, s->x, s->nrm, s->w,
                       static_cast<double*>(P.rec));  // no pass runs yet
    SDBIE_LAUNCHED();
    static_assert(kScanBlocks * 8 * sizeof(double) <= kTile * kRecBytes, "the block results fit one tile's records");
    hipLaunchKernelGGL(k_morton, dim3((unsigned)((P.npow2 + 255) / 256)), dim3(256), 0, st, n, P.npow2, s->x,
                       static_cast<const double*>(P.rec), stage, P.keys);
    SDBIE_LAUNCHED();
    sort_keys(P.keys, P.npow2, st);
    StageArgs a;
    a.n = n;
    a.npad = P.npad;
    a.keys = P.keys;
    a.x = s->x;
    a.nrm = s->nrm;
    a.w = s->w;
    a.bb = stage + 2;
    a.perm = P.perm;
    a.xs = P.x;
    a.ns = P.nrm;
    a.ws = P.w;
    a.wn = P.wn;
    a.px = P.px;
    a.pn = P.pn;
    a.pw = P.pw;
    a.px32 = P.px32;
    a.boxes = P.boxes;
    a.uboxes = P.uboxes;
    hipLaunchKernelGGL(k_stage, dim3((unsigned)P.ntiles), dim3(kTile), 0, st, a);
    SDBIE_LAUNCHED();
    // cutoffs with a relative margin of 1e-6 (the far kernels assume rho >= rho_cut)
    const double rc64 = SDBIE_RHO_CUT_STOKES_F64 * P.delta * (1.0 + 1e-6);
    const double rc32 = SDBIE_RHO_CUT_STOKES_F32 * P.delta * (1.0 + 1e-6);
    const bool lists = P.sym[0].items != nullptr;
    if (lists && P.ntiles > kSymMaxTiles) throw Error(SDBIE_ERR_ARG, "internal: symmetric lists of too many tiles");
    hipLaunchKernelGGL(k_mask_rows, dim3((unsigned)(P.ntiles > kRedBlocks ? P.ntiles : kRedBlocks)), dim3(256), 0, st,
                       P.ntiles, n, (const double*)P.boxes, rc64, rc32, P.mask64, P.mask32,
                       reinterpret_cast<unsigned long long*>(stage + 10), lists ? P.sym_rows : nullptr,
                       static_cast<int32_t*>(P.rec), (const double*)P.w, P.red);
    SDBIE_LAUNCHED();
    if (lists) {
        build_symmetric_lists(P, reinterpret_cast<int32_t*>(stage + 12), st);
    } else {
        hipLaunchKernelGGL(k_area, dim3(1), dim3(256), 0, st, (const double*)P.red, stage + 8);
        SDBIE_LAUNCHED();
    }
    struct {
        int32_t flag[2];
        double pad[7], area, pad9;
        unsigned long long near[2];
        int32_t blocks[8];
    } h;
    static_assert(sizeof(h) == 16 * sizeof(double), "the staging scalars (solver.h)");
    SDBIE_HIP(hipMemcpyAsync(&h, stage, sizeof(h), hipMemcpyDeviceToHost, st));
    SDBIE_HIP(hipStreamSynchronize(st));
    if (h.flag[0]) throw Error(SDBIE_ERR_NONFINITE, "non-finite node coordinates, normals or weights");
    if (h.flag[1]) throw Error(SDBIE_ERR_ARG, "node coordinates must not exceed 1e15 in magnitude");
    if (!(h.area > 0.0)) throw Error(SDBIE_ERR_ARG, "the quadrature weights sum to zero");
    P.near_pairs64 = (double)h.near[0];
    P.near_pairs32 = (double)h.near[1];
    P.area = h.area;
    for (int k = 0; lists && k < 3; ++k) P.sym[k].nblocks = h.blocks[k];
}

}  // namespace sdbie
