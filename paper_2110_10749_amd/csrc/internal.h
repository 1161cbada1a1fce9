// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <stdexcept>
#include <string>

#include "../../include/sdbie.h"

namespace sdbie {

// Sum over a wave, every lane the same: lanes 32, 16, 8, 4, 2 and 1 apart.  The last
// four steps are DPP moves; after the step of 8, lane l +- 4 of a row hold the same
// value, so the direction of the rotation by 4 does not matter.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
    v = dpp_add<0x128>(v);        // row_ror:8
    v = dpp_add<0x124>(v);        // row_ror:4
    v = dpp_add<0x4e>(v);         // quad_perm [2, 3, 0, 1]
    return dpp_add<0xb1>(v);      // quad_perm [1, 0, 3, 2]
}

// Error carried inside the library; converted to a status code at the C ABI.
struct Error : std::runtime_error {
    int code;
    Error(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

#define SDBIE_HIP(call)                                                                     \
    do {                                                                                    \
        hipError_t e_ = (call);                                                             \
        if (e_ != hipSuccess)                                                               \
            throw ::sdbie::Error(SDBIE_ERR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define SDBIE_LAUNCHED() SDBIE_HIP(hipGetLastError())

constexpr int kTPB = 256;        // threads per block of the pair kernels (4 waves)
constexpr int kTile = 256;       // sources staged in LDS per tile
constexpr int kMaxSplit = 64;    // source splits of one pair pass
constexpr int64_t kMaxNodes = (int64_t)1 << 23;  // the tile-pair masks grow as (n/256)^2 bytes
constexpr int kNearUnit = 64;    // sources per work unit of the near-field kernel
constexpr int kRecBytes = 128;   // largest per-source record of a pair pass
// bytes of source records per unrolled step of the pair loops
#ifndef SDBIE_GROUP_BYTES_F32
#define SDBIE_GROUP_BYTES_F32 128
#endif
// far- and near-field blocks of a pass in one launch (1) or in two (0)
#ifndef SDBIE_ONE_LAUNCH
#define SDBIE_ONE_LAUNCH 1
#endif
// float far-field records through LDS (1) or the scalar cache (0)
#ifndef SDBIE_FAR_LDS
#define SDBIE_FAR_LDS 1
#endif
#ifndef SDBIE_GROUP_BYTES_F64
#define SDBIE_GROUP_BYTES_F64 128
#endif
constexpr int kMaxRestart = 1000; // largest GMRES restart length of a plan
// symmetric passes (sym_body): tile pairs per block at most, parts a tile pair
// is cut into at most, blocks a pass aims for, and the bits of an item's steps:
// 16 row rotations, whether the pair may hold pairs within the cutoff, and the
// rotations of a tile against itself
constexpr int kSymChunk = 8;
constexpr int kSymParts = 16;
// tiles up to which a plan holds the work lists: 524288 nodes, 14.7 GB of lists and
// slots.  Staging sizes its arrays by it and ranks far pairs in the records' memory.
#ifndef SDBIE_SYM_MAX_TILES
#define SDBIE_SYM_MAX_TILES 2048
#endif
constexpr int kSymMaxTiles = SDBIE_SYM_MAX_TILES;
static_assert(kSymMaxTiles % 256 == 0, "whole groups of 64 tiles, and rows per thread of a 256-thread block");
static_assert((int64_t)kSymMaxTiles * sizeof(int32_t) <= (int64_t)kTile * kRecBytes, "T^2 ranks fit T tiles' records");
#ifndef SDBIE_SYM_TARGET
#define SDBIE_SYM_TARGET 16384
#endif
#ifndef SDBIE_SYM_PARTS
#define SDBIE_SYM_PARTS 4096
#endif
constexpr int kSymAll = 0xffff, kSymNear = 0x10000, kSymSelf = 0x03ff;
constexpr size_t kSymSlotBytes = (size_t)3 * kTile * sizeof(double);
#ifndef SDBIE_SPLIT_TARGET
#define SDBIE_SPLIT_TARGET 4096      // far-field blocks a pass kernel aims for (the near-field blocks double them)
#endif
// accepted input range: |coordinates| <= kMaxCoord, delta in [kMinDelta, kMaxCoord],
// so every pair distance squared is a normal number in float and double
constexpr double kMaxCoord = 1e15;
constexpr double kMinDelta = 1e-15;
constexpr int kRedBlocks = 512;  // blocks of the deterministic reductions
// columns up to which a Krylov step runs the fused Gram-Schmidt kernels; past
// that the redundant reductions of every block would take longer than the
// launches they save
constexpr int kFuseCols = 64;
// host memory of a solve (doubles): what the fused kernels write for the host
enum : int {
    kHostE = 0, kHostH1 = kFuseCols, kHostH2 = 2 * kFuseCols, kHostNorm = 3 * kFuseCols,
    kHostDot = 3 * kFuseCols + 8, kHostDoubles = kHostDot + kRedBlocks,
};
// most bytes of partial slots beyond the one-direction passes' that a plan of few
// tiles takes for the slots of its symmetric passes
constexpr size_t kMinPartial = (size_t)12 << 20;

// Pair-sum passes --------------------------------------------------------------
// Laplace pass:  out_i = base_i + c_dl * sum_j w_j (q_j - sub*q_i)(D.n_j) k2
//                               + c_sl * sum_j w_j g_j k1 + comp * cw_i
// Stokes pass:   out_i = base_i + c_dl * sum_j w_j ((u_j - sub*u_i).D)(D.n_j) D k4
//                               + c_sl * sum_j w_j [f_j k1 + D (D.f_j) k3]
//                               + comp * n_i
// where the Stokes single-layer density is f = sl_dens, or beta * P_tau u
// when slip_beta != 0 (computed on the fly from the double-layer density).
struct PassDesc {
    bool dl = false, sl = false, sub = false;
    double c_dl = 0.0, c_sl = 0.0;
    const double* dl_dens = nullptr;  // sorted
    const double* sl_dens = nullptr;  // sorted
    double slip_beta = 0.0;           // Stokes only
    const double* base = nullptr;     // sorted, [n] or [3][n], added to the result (nullable)
    double base_scale = 1.0;
    // completion (nullable): comp_scale (comp_a . comp_b) added to every node
    // (Laplace) or times its normal (Stokes).  The dot product's block partials
    // are taken by the packing kernel and summed by the epilogue.
    const double* comp_a = nullptr;
    const double* comp_b = nullptr;
    double comp_scale = 0.0;
    // the density in the caller's order (nullable): gathered into dl_dens /
    // sl_dens (gather_dst, all components) by the packing kernel
    const double* gather_src = nullptr;
    double* gather_dst = nullptr;
    const double* add_const = nullptr; // host double[3] added to every node (nullable)
    double* out = nullptr;            // sorted, or original order when scatter
    bool scatter = false;             // write out[perm[i]] instead of out[i]
    bool mixed = false;
    // transposed sums (adjoint)
    bool unit_src_weight = false;     // sources enter with weight 1 instead of w_j
    bool target_weight = false;       // the pair sum is multiplied by the target's w_i
    bool target_normal = false;       // double layer contracted with the target's normal (transposed DL)
    const double* dl_target = nullptr;  // target density of the subtracted double layer (default dl_dens)
};

// Position-gradient pass of the adjoint: for every pair (i, j),
//   g_ij = grad_D [lam1_i T1_ij + lam2_i . T2_ij],  D = x_i - x_j,
//   T1_ij = c_l w_j (p_j - p_i)(D.n_j) K2 + (mu/K) c_l w_j v_j K1,
//   T2_ij = c_s w_j ((u_j - u_i).D)(D.n_j) D K4 + c_v w_j [f_j K1 + D (D.f_j) K3],
// with c_l = 1/(4 pi), c_s = -3/(4 pi), c_v = 1/(8 pi mu); the pass writes
// out_m = -sum_j g_mj + sum_i g_im (derivative of -lam^T F w.r.t. x_m).
struct GradDesc {
    double mu, K;
    const double *p, *v, *u, *f, *lam1, *lam2;  // sorted, stride n
    double* out;                                // sorted [3][n]
};

// Work of a symmetric pass: the tile pairs {a <= b}, each cut into parts, as
// items (a, b, reverse slot, steps); blocks of items of one target tile, near
// pairs first (they take longest); the first forward slot (one per block) of
// each target tile and the first reverse slot (one per part of a pair a < b,
// column by column) of each source tile.
// The far-only set holds the far tile pairs alone, kSymChunk to a block; its
// passes evaluate the near tile pairs in one-direction near-field blocks.
// FP64 coupled solves and adjoints run on it: their inexact interface products
// make the result within tol_ddm a function of every rounding of the pair
// sums (the same solve with the near pairs summed in another order moves by
// 1e-8 at the default tolerance), and these sums keep their order.
enum : int { kSymF64 = 0, kSymF32 = 1, kSymFar64 = 2 };
struct SymSet {
    int nblocks = 0, parts = 1;
    int32_t* items = nullptr;      // [nitems][4]
    int32_t* blocks = nullptr;     // [nblocks][3]: first item, item count, forward slot
    int32_t* fwd_start = nullptr;  // [ntiles + 1]
    int32_t* rev_start = nullptr;  // [ntiles + 1]
    double* fwd = nullptr;         // [nblocks][C][kTile] forward partials of the target tile, C <= 3
    void* rev = nullptr;           // [slots][C][kTile doubles] reverse partials of the source tile (rev_slot)
};
constexpr int kSymRowInts = 16;

struct Plan {
    int64_t n = 0;
    int max_restart = 0;
    double delta = 0.0;
    double area = 0.0;  // sum of weights
    // sorted node data (double)
    double* x = nullptr;    // [3][n]
    double* nrm = nullptr;  // [3][n]
    double* w = nullptr;    // [n]
    double* wn = nullptr;   // [3][n] w_j n_j
    // sorted node data padded to whole tiles of kTile nodes (pair-kernel sources;
    // padding nodes sit far outside the body with zero weight and normal)
    int64_t npad = 0;       // ntiles * kTile
    int ntiles = 0;
    double* px = nullptr;   // [3][npad]
    double* pn = nullptr;   // [3][npad]
    double* pw = nullptr;   // [npad]
    float* px32 = nullptr;  // [3][npad], each node minus the centre of its tile's box
    double* boxes = nullptr;   // [ntiles][6] min/max per axis
    double* uboxes = nullptr;  // [npad / kNearUnit][6]: the same per near-field unit of sources
    uint8_t* mask64 = nullptr; // [ntiles][ntiles]: 1 if the tile pair may hold a pair with rho < double cutoff
    uint8_t* mask32 = nullptr; // [ntiles][ntiles]: same with the float cutoff
    int32_t* perm = nullptr;  // sorted index -> caller index
    uint64_t* keys = nullptr; // sort scratch, [npow2]
    int64_t npow2 = 0;
    // scratch
    int nsplit = 0;             // source splits of a pair pass (choose_splits(n) or fewer)
    int max_comps = 6;          // components a pass may write per slot (the partial buffer's C)
    double* partial = nullptr;  // [2 * nsplit][C][n], C <= max_comps: far splits then near splits
    void* rec = nullptr;        // per-pass source records, [npad][kRecBytes]
    double* red = nullptr;      // reduction partials [kRedBlocks * 64]
    double* scal = nullptr;     // small device scalars / columns [256]
    double* vecs = nullptr;     // general work vectors, kNumVec x [3][n]
    double* basis_in = nullptr;   // inner GMRES basis [(max_restart+1)][3n]
    double* basis_out = nullptr;  // outer GMRES basis [(max_restart+1)][n]
    double* image_out = nullptr;  // local solutions (p, u) and right-hand sides (b_D, b_S) of each outer
                                  // basis vector [(max_restart+1)][8n]
    double* basis_rc = nullptr;   // recycled inner basis (deflation space) [(max_restart+1)][3n]
    double* host_pinned = nullptr;  // [kHostDoubles] host memory the kernels write to (during a solve, see Ctx)
    // (target, source) pairs of real nodes in the near tile pairs (double, float masks)
    double near_pairs64 = 0.0, near_pairs32 = 0.0;
    // target-source symmetric passes (for the pass kinds whose SDBIE_SYM_* bit is
    // set in `symmetric`): double, float, and the double far pairs alone
    int symmetric = SDBIE_SYM_DEFAULT;
    SymSet sym[3];
    bool far_only64 = false;         // double passes take sym[2] and the near-field blocks (see SymSet)
    void* sym_fwd_mem = nullptr;     // the workspace regions the slots are placed in (stage.hip), besides `partial`
    void* sym_rev_mem = nullptr;
    size_t partial_bytes = 0, sym_fwd_bytes = 0;
    int32_t* sym_rows = nullptr;     // staging scratch [ntiles][kSymRowInts]
    // bookkeeping for info
    int64_t applies_fp64 = 0, applies_mixed = 0;
    double pairs = 0.0;
    double* vec(int k) const { return vecs + (size_t)k * 3 * n; }
};

constexpr int kNumVec = 31;
constexpr int kImageStride = 8;  // doubles per node of one image-basis slot: p, u, b_D, b_S

// parts a tile pair of a symmetric pass is cut into on a surface of nt tiles
int sym_parts(int64_t nt);
size_t workspace_bytes(int64_t n, int max_restart);
void carve_workspace(Plan& P, void* ws);
// layer applies only (no solver vectors), at most nsplit_cap source splits and
// three components per partial slot: bytes, and the carve (which also sets
// *in, a [3][n] buffer for the gathered density)
size_t layer_workspace_bytes(int64_t n, int nsplit_cap);
void carve_layer_workspace(Plan& P, void* ws, int nsplit_cap, double** in);
// the layer sums of the C ABI on a staged plan; `in` receives the density in
// staged order ([n] or [3][n])
void apply_laplace_layer(Plan& P, sdbie_layer layer, const double* dens, double* out, sdbie_precision prec,
                         hipStream_t st, double* in);
void apply_stokes_layer(Plan& P, double mu, sdbie_layer layer, const double* dens, double* out,
                        sdbie_precision prec, hipStream_t st, double* in);

// allocation-free layer sum (noalloc.hip): stages s into the library's static
// device array and applies the Stokes layer
void stokes_layer_apply_static(const sdbie_surface* s, double mu, sdbie_layer layer, const double* dens,
                               double* out, sdbie_precision prec, hipStream_t st);

// kernels (pair_kernels.hip) ----------------------------------------------------
void launch_laplace_pass(const Plan& P, const PassDesc& d, hipStream_t s);
void launch_stokes_pass(const Plan& P, const PassDesc& d, hipStream_t s);
void launch_grad_pass(const Plan& P, const GradDesc& g, hipStream_t s);
int choose_splits(int64_t n);

// kernel timing (profile.hip)
int prof_variant(int family, bool mixed, int code, int part);
struct ProfScope {
    ProfScope(int variant, double pairs, hipStream_t s);
    ~ProfScope();
    hipStream_t s_;
    long idx_ = -1;
};

// staging (stage.hip) --------------------------------------------------------------
void stage_surface(Plan& P, const sdbie_surface* s, hipStream_t st);

// vector kernels (blas.hip) ----------------------------------------------------------
// deterministic dot product sum_i a_i b_i (len elements) -> device scalar *out
void dev_dot(const Plan& P, const double* a, const double* b, int64_t len, double* out, hipStream_t s);
// dots of w against k columns of V (column stride ld) -> out[0..k-1]
void dev_multidot(const Plan& P, const double* V, int64_t ld, int k, const double* w, int64_t len,
                  double* out, hipStream_t s);
// One Krylov step: w is orthogonalised against k columns V twice (CGS2; leading
// dimension len) and next = w / ||w||; with kr > 0 first against the deflation
// space Vr (kr + 1 columns, rotations rot on the device).  k, kr + 1 <= kFuseCols.
// After a stream synchronisation host_pinned holds the coefficients (kHostE,
// kHostH1, kHostH2) and the squared norm (kHostNorm).
void dev_cgs2(const Plan& P, const double* Vr, int kr, const double* rot, const double* V, int k, double* w,
              double* next, int64_t len, hipStream_t s);
// dot product on the host (synchronises the stream), summed in dev_dot's order
double dev_dot_host(const Plan& P, const double* a, const double* b, int64_t len, hipStream_t s);
// w -= sum_j h[j] V_j  (h on device)
void dev_multi_axpy_sub(const double* V, int64_t ld, int k, const double* h, double* w, int64_t len,
                        hipStream_t s);
// x += sum_j y[j] V_j  (y on device)
void dev_multi_axpy_add(const double* V, int64_t ld, int k, const double* y, double* x, int64_t len,
                        hipStream_t s);
void dev_axpby(double a, const double* x, double b, const double* y, double* out, int64_t len, hipStream_t s);
void dev_scale(double a, const double* x, double* out, int64_t len, hipStream_t s);
void dev_fill(double v, double* out, int64_t len, hipStream_t s);
void dev_add_scaled_scalar(double* x, const double* dscal, double scale, int64_t len, hipStream_t s);
// out = u.n (per node)
void dev_normal_component(const Plan& P, const double* u, double* out, hipStream_t s);
// f = -p n + beta (u - (u.n) n) + f_extra   (u, f_extra nullable)
void dev_traction(const Plan& P, const double* p, const double* u, double beta, const double* f_extra,
                  double* f, hipStream_t s);
// sorted <-> caller order
void dev_gather(const Plan& P, const double* src, double* dst, int comps, hipStream_t s);
void dev_scatter(const Plan& P, const double* src, double* dst, int comps, hipStream_t s);
// adjoint helpers (see blas.hip)
void dev_adj_darcy(const Plan& P, const double* tn, const double* lam, const double* dl1, const double* sum,
                   double* out, hipStream_t s);
void dev_adj_stokes(const Plan& P, const double* lam, const double* m0, const double* m1, const double* m2,
                    const double* tns, const double* sv, const double* flux, double beta, double* out, hipStream_t s);
void dev_scalar_normal(const Plan& P, const double* sv, double scale, double* out, hipStream_t s);
void dev_axpy_w(const Plan& P, double* x, const double* d, double scale, hipStream_t s);
void dev_adj_rhs(const Plan& P, const double e[3], double beta, double* gp, double* gu, hipStream_t s);

// host-side helpers
// eigenvalues of an upper Hessenberg matrix (n x n, row-major, overwritten); false if the QR iteration stalls
bool hessenberg_eigenvalues(int n, double* A, double* wr, double* wi);

}  // namespace sdbie
