// Surface staging: spatial (Morton) order and the sorted node copies.
//
// The pair kernels give each wave 64 consecutive targets; sorting the nodes
// along a Morton (Z-order) curve makes those 64 targets spatial neighbours,
// so the near-field branch (rho < rho_cut) is taken by few waves per source
// and the rest run the plain far-field kernel.
//
// Steps (all on the device): bounding box (min/max reduction), 30-bit Morton
// key per node (10 bits per axis), key<<32 | index sorted by a bitonic network
// over the next power of two (padding keys = UINT64_MAX; keys are unique, so
// the order is deterministic), then gather of x, n, w into sorted double
// arrays and the weighted normals w n; copies padded to whole tiles of kTile
// nodes for the pair kernels; per-tile bounding boxes; a float copy of the
// coordinates in the frame of each node's tile; and the near-field masks of
// tile pairs (box distance below rho_cut delta, one mask for the double cutoff
// and one for the float cutoff).

#include "smoothing_coeffs.h"
#include "solver.h"

namespace sdbie {
namespace {

__global__ __launch_bounds__(256) void k_bbox(int64_t n, const double* __restrict__ x, double* __restrict__ out) {
    // one block per axis: out[2c] = min, out[2c+1] = max
    __shared__ double smin[256], smax[256];
    const int c = blockIdx.x;
    double lo = INFINITY, hi = -INFINITY;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double v = x[c * n + i];
        lo = fmin(lo, v);
        hi = fmax(hi, v);
    }
    smin[threadIdx.x] = lo;
    smax[threadIdx.x] = hi;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[2 * c] = smin[0];
        out[2 * c + 1] = smax[0];
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

__global__ void k_morton(int64_t n, int64_t npow2, const double* __restrict__ x, const double* __restrict__ bb,
                         uint64_t* __restrict__ keys) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
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

__global__ void k_bitonic(uint64_t* __restrict__ keys, int64_t npow2, int64_t j, int64_t k) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npow2) return;
    const int64_t l = i ^ j;
    if (l > i) {
        const uint64_t a = keys[i], b = keys[l];
        const bool up = (i & k) == 0;
        if ((a > b) == up) {
            keys[i] = b;
            keys[l] = a;
        }
    }
}

__global__ void k_stage(int64_t n, const uint64_t* __restrict__ keys, const double* __restrict__ x,
                        const double* __restrict__ nrm, const double* __restrict__ w, int32_t* __restrict__ perm,
                        double* __restrict__ xs, double* __restrict__ ns, double* __restrict__ wsrt,
                        double* __restrict__ wn) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int64_t o = (int64_t)(keys[k] & 0xffffffffull);
    perm[k] = (int32_t)o;
    const double wk = w[o];
    wsrt[k] = wk;
    for (int c = 0; c < 3; ++c) {
        const double xv = x[c * n + o], nv = nrm[c * n + o];
        xs[c * n + k] = xv;
        ns[c * n + k] = nv;
        wn[c * n + k] = wk * nv;
    }
}

// padded copies for the pair kernels: nodes k >= n sit at a point `far`
// outside the bounding box (10 extents away) with zero weight and normal.
__global__ void k_pad(int64_t n, int64_t npad, const double* __restrict__ xs, const double* __restrict__ ns,
                      const double* __restrict__ ws, const double* __restrict__ bb, double* __restrict__ px,
                      double* __restrict__ pn, double* __restrict__ pw) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npad) return;
    const double ext = fmax(fmax(bb[1] - bb[0], bb[3] - bb[2]), bb[5] - bb[4]);
    for (int c = 0; c < 3; ++c) {
        const double xv = k < n ? xs[c * n + k] : bb[2 * c + 1] + 10.0 * ext + 1.0;
        px[c * npad + k] = xv;
        pn[c * npad + k] = k < n ? ns[c * n + k] : 0.0;
    }
    pw[k] = k < n ? ws[k] : 0.0;
}

// float coordinates in the frame of their tile: minus the centre of the tile's
// box (every tile holds at least one real node, so the centre is finite).  The
// kernels see coordinates only through differences x_i - x_j, formed after
// moving the targets into the source tile's frame, so the rounding of a float
// coordinate is set by the tile's extent, not by the body's or by the
// distance from the origin.
__global__ void k_frame32(int64_t npad, const double* __restrict__ px, const double* __restrict__ boxes,
                          float* __restrict__ px32) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npad) return;
    const double* b = boxes + (k / kTile) * 6;
    for (int c = 0; c < 3; ++c) px32[c * npad + k] = (float)(px[c * npad + k] - 0.5 * (b[2 * c] + b[2 * c + 1]));
}

// bounding box of each group of W consecutive (sorted) real nodes (empty:
// +inf / -inf for a group of padding only); one block of W threads per group
template <int W>
__global__ __launch_bounds__(W) void k_boxes(int64_t n, const double* __restrict__ xs, double* __restrict__ boxes) {
    __shared__ double sh[6][W];
    const int64_t k = (int64_t)blockIdx.x * W + threadIdx.x;
    for (int c = 0; c < 3; ++c) {
        const double v = k < n ? xs[c * n + k] : NAN;
        sh[2 * c][threadIdx.x] = k < n ? v : INFINITY;
        sh[2 * c + 1][threadIdx.x] = k < n ? v : -INFINITY;
    }
    __syncthreads();
    for (int s = W / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int c = 0; c < 3; ++c) {
                sh[2 * c][threadIdx.x] = fmin(sh[2 * c][threadIdx.x], sh[2 * c][threadIdx.x + s]);
                sh[2 * c + 1][threadIdx.x] = fmax(sh[2 * c + 1][threadIdx.x], sh[2 * c + 1][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) boxes[(int64_t)blockIdx.x * 6 + threadIdx.x] = sh[threadIdx.x][0];
}

// mask[b][t] = 1 when the boxes of tiles b and t are closer than the cutoff.
// cnt[0], cnt[1] += the (target, source) pairs of real nodes in the near tile
// pairs of each precision (integer sums: exact in any order).
__global__ void k_near_masks(int nt, int64_t n, const double* __restrict__ boxes, double rc64, double rc32,
                             uint8_t* __restrict__ m64, uint8_t* __restrict__ m32,
                             unsigned long long* __restrict__ cnt) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long c64 = 0, c32 = 0;
    if (idx < (int64_t)nt * nt) {
        const int64_t b = idx / nt, t = idx % nt;
        const double* A = boxes + b * 6;
        const double* B = boxes + t * 6;
        double d2 = 0.0;
        for (int c = 0; c < 3; ++c) {
            const double gap = fmax(0.0, fmax(A[2 * c] - B[2 * c + 1], B[2 * c] - A[2 * c + 1]));
            d2 += gap * gap;
        }
        const bool n64 = d2 < rc64 * rc64, n32 = d2 < rc32 * rc32;
        m64[idx] = n64 ? 1 : 0;
        m32[idx] = n32 ? 1 : 0;
        const int64_t rb = n - b * kTile < kTile ? n - b * kTile : kTile;
        const int64_t rt = n - t * kTile < kTile ? n - t * kTile : kTile;
        const unsigned long long pr = (unsigned long long)(rb * rt);
        c64 = n64 ? pr : 0;
        c32 = n32 ? pr : 0;
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

// Work lists of the symmetric passes, from the near masks, in three kernels:
// counts of each mask row, their prefix sums (one block), and the items and
// blocks of each row.  Blocks hold as many pairs as leave about
// SDBIE_SYM_TARGET of them for each kind of pair (at most kSymChunk while the
// forward slots have room): with 8 pairs to a block the 2200 pairs of n = 17070
// made 343 blocks for 256 CUs.

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

__global__ __launch_bounds__(256) void k_list_rows(int T, const uint8_t* __restrict__ m64,
                                                   const uint8_t* __restrict__ m32, int32_t* __restrict__ rows,
                                                   int32_t* __restrict__ colrank) {
    __shared__ int sh[4];
    const int a = blockIdx.x;
    int cnt[5] = {0, 0, 0, 0, 0};
    for (int b0 = 0; b0 < T; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const bool in = b < T;
        const bool n64 = in && m64[(int64_t)a * T + b], n32 = in && m32[(int64_t)a * T + b];
        int t;
        block_rank(in && b > a && n64, sh, t);
        cnt[kRowNear64] += t;
        block_rank(in && b > a && !n64, sh, t);
        cnt[kRowFar64] += t;
        // the masks are symmetric: row a, b < a, is the far-only column of source tile a
        const bool cf = in && b < a && !n64;
        const int r = block_rank(cf, sh, t);
        if (cf) colrank[(int64_t)a * T + b] = cnt[kRowColFar64] + r;
        cnt[kRowColFar64] += t;
        block_rank(in && b != a && n32, sh, t);
        cnt[kRowNear32] += t;
        block_rank(in && b > a && !n32, sh, t);
        cnt[kRowFar32] += t;
    }
    if (threadIdx.x < 5) rows[(int64_t)a * kSymRowInts + threadIdx.x] = cnt[threadIdx.x];
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
};

constexpr int kScanRows = 8;  // rows per thread of the scan (2048 tiles)

// exclusive prefix sums over the rows of v[0..kScanRows) (thread-consecutive), total over all
__device__ __forceinline__ int block_scan(int (&v)[kScanRows], int* sh) {
    int s = 0;
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
        const int t = v[i];
        v[i] = s;
        s += t;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const int t = (int)threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    const int base = threadIdx.x ? sh[threadIdx.x - 1] : 0, total = sh[255];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] += base;
    return total;
}

__global__ __launch_bounds__(256) void k_list_scan(ListArgs A) {
    __shared__ int sh[256];
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

// Enqueues the list kernels; the block counts arrive in out[0..2] (device).
// Forward and reverse slots of several parts to a pair share the partial
// buffer of the one-direction passes; of one part the reverse slots have their
// own region, and the forward ones take the larger of the buffer and sym_fwd.
void build_symmetric_lists(Plan& P, int32_t* out, hipStream_t st) {
    const int T = P.ntiles;
    if (T > 256 * kScanRows) throw Error(SDBIE_ERR_ARG, "internal: symmetric lists of too many tiles");
    const int64_t pairs = (int64_t)T * (T - 1) / 2;
    ListArgs A;
    A.T = T;
    A.mask[0] = P.mask64;
    A.mask[1] = P.mask32;
    A.rows = P.sym_rows;
    A.colrank = static_cast<const int32_t*>(P.rec);  // T^2 ints; no pass runs yet
    A.out = out;
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
    hipLaunchKernelGGL(k_list_rows, dim3((unsigned)T), dim3(256), 0, st, T, (const uint8_t*)P.mask64,
                       (const uint8_t*)P.mask32, P.sym_rows, static_cast<int32_t*>(P.rec));
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_list_scan, dim3(1), dim3(256), 0, st, A);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_list_fill, dim3((unsigned)T), dim3(256), 0, st, A);
    SDBIE_LAUNCHED();
}

}  // namespace

void stage_surface(Plan& P, const sdbie_surface* s, hipStream_t st) {
    const int64_t n = P.n;
    // finite check of the node data first (Morton keys of NaN are meaningless)
    // flags and counters are cleared by a fill kernel, not a memset node (the
    // staging of the allocation-free entry point may sit in a captured stream)
    int* flag = reinterpret_cast<int*>(P.scal + kScalStage);
    dev_fill(0.0, P.scal + kScalStage, 1, st);  // two ints
    dev_check_finite(s->x, 3 * n, kMaxCoord, flag, st);
    dev_check_finite(s->nrm, 3 * n, HUGE_VAL, flag, st);
    dev_check_finite(s->w, n, HUGE_VAL, flag, st);
    int hflag[2] = {0, 0};
    SDBIE_HIP(hipMemcpyAsync(hflag, flag, sizeof(hflag), hipMemcpyDeviceToHost, st));
    SDBIE_HIP(hipStreamSynchronize(st));
    if (hflag[0]) throw Error(SDBIE_ERR_NONFINITE, "non-finite node coordinates, normals or weights");
    if (hflag[1]) throw Error(SDBIE_ERR_ARG, "node coordinates must not exceed 1e15 in magnitude");

    double* bb = P.scal + kScalStage + 2;
    hipLaunchKernelGGL(k_bbox, dim3(3), dim3(256), 0, st, n, s->x, bb);
    SDBIE_LAUNCHED();
    const unsigned nb = (unsigned)((P.npow2 + 255) / 256);
    hipLaunchKernelGGL(k_morton, dim3(nb), dim3(256), 0, st, n, P.npow2, s->x, (const double*)bb, P.keys);
    SDBIE_LAUNCHED();
    for (int64_t k = 2; k <= P.npow2; k <<= 1)
        for (int64_t j = k >> 1; j > 0; j >>= 1) {
            hipLaunchKernelGGL(k_bitonic, dim3(nb), dim3(256), 0, st, P.keys, P.npow2, j, k);
            SDBIE_LAUNCHED();
        }
    hipLaunchKernelGGL(k_stage, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, (const uint64_t*)P.keys,
                       s->x, s->nrm, s->w, P.perm, P.x, P.nrm, P.w, P.wn);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_pad, dim3((unsigned)((P.npad + 255) / 256)), dim3(256), 0, st, n, P.npad,
                       (const double*)P.x, (const double*)P.nrm, (const double*)P.w, (const double*)bb, P.px, P.pn,
                       P.pw);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL((k_boxes<kTile>), dim3((unsigned)P.ntiles), dim3(kTile), 0, st, n, (const double*)P.x,
                       P.boxes);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL(k_frame32, dim3((unsigned)((P.npad + 255) / 256)), dim3(256), 0, st, P.npad,
                       (const double*)P.px, (const double*)P.boxes, P.px32);
    SDBIE_LAUNCHED();
    hipLaunchKernelGGL((k_boxes<kNearUnit>), dim3((unsigned)(P.npad / kNearUnit)), dim3(kNearUnit), 0, st, n,
                       (const double*)P.x, P.uboxes);
    SDBIE_LAUNCHED();
    // cutoffs with a relative margin of 1e-6 (the far kernels assume rho >= rho_cut)
    const double rc64 = SDBIE_RHO_CUT_STOKES_F64 * P.delta * (1.0 + 1e-6);
    const double rc32 = SDBIE_RHO_CUT_STOKES_F32 * P.delta * (1.0 + 1e-6);
    const int64_t nt2 = (int64_t)P.ntiles * P.ntiles;
    unsigned long long* cnt = reinterpret_cast<unsigned long long*>(P.scal + kScalStage + 10);
    dev_fill(0.0, P.scal + kScalStage + 10, 2, st);  // two 64-bit counters (all-zero bits)
    hipLaunchKernelGGL(k_near_masks, dim3((unsigned)((nt2 + 255) / 256)), dim3(256), 0, st, P.ntiles, n,
                       (const double*)P.boxes, rc64, rc32, P.mask64, P.mask32, cnt);
    SDBIE_LAUNCHED();
    const bool lists = P.sym[0].items != nullptr;
    if (lists) build_symmetric_lists(P, reinterpret_cast<int32_t*>(P.scal + kScalStage + 12), st);
    dev_dot(P, P.w, nullptr, n, P.scal + kScalStage + 8, st);
    struct {
        double area, pad;
        unsigned long long near[2];
        int32_t blocks[8];
    } h;
    static_assert(sizeof(h) == 8 * sizeof(double), "area (8), near-pair counts (10, 11), list counts (12 ..)");
    SDBIE_HIP(hipMemcpyAsync(&h, P.scal + kScalStage + 8, sizeof(h), hipMemcpyDeviceToHost, st));
    SDBIE_HIP(hipStreamSynchronize(st));
    P.near_pairs64 = (double)h.near[0];
    P.near_pairs32 = (double)h.near[1];
    P.area = h.area;
    for (int k = 0; lists && k < 3; ++k) P.sym[k].nblocks = h.blocks[k];
    if (!(P.area > 0.0)) throw Error(SDBIE_ERR_ARG, "the quadrature weights sum to zero");
}

}  // namespace sdbie
