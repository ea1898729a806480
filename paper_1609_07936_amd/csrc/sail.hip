// sail.hip -- gfx950 kernels and C ABI for the simulated-annealing inverse
// Laplace transform (Lutsyshyn & Astrakharchik, arXiv:1609.07936).
//
// Device layout (one problem, N_w walkers, N_omega bins, N_tau times):
//   * The model kernel is separable, K(omega_j, tau_i) = c_i e^{-omega_j tau_i}
//     (c_i = d_omega / 2pi for bin-centre sampling, the bin-integral factor for
//     the exact bin integral of Eq. correlation-model).  The walkers carry
//     Phi_i = F_i / c_i, so the data become Phit_i = F_i / c_i and the weights
//     wh_i = c_i^2 / sigma_i^2; chi^2 is unchanged.
//   * The weighted columns sqrt(wh_i) e^{-omega_j tau_i} of all bins lie, to
//     rounding, in a space of few dimensions (16 for the benchmark's 512 bins
//     and 128 times): a Laplace kernel's singular values fall geometrically.
//     The host builds an orthonormal basis of it from a sample of columns, the
//     device projects all of them, the sweep carries each
//     walker's coordinates phi of sqrt(wh) Phi in that basis, and sums over
//     tau become sums over the basis.
//   * A walker occupies G lanes of a wavefront; lane c holds chunk c mod 4 of
//     phi in registers (a quarter of it where the basis is wide).  The residue change is taken from its expansion, whose
//     only sum that needs the walker is sum_i w_i Phi_i s_i = phi . sigma with
//     sigma = dp C_p + ds C_s (C_j: column j in the basis; four chunk sums and
//     a two-step butterfly, so every lane ends with the same bits and takes the
//     same accept decision, whatever G is); the walker-independent sums come
//     from per-bin and pair-sum tables, and a commit is phi = r phi + sigma.
//   * Spectra live in HBM as b_j with a_j = g b_j (a lazy scale g per walker),
//     so a move touches two coefficients instead of N_omega; the scale is folded
//     back at resync.  While a sweep runs they sit in LDS where they fit; else
//     lane c of a walker owns the spectrum accesses of a batch's proposal c.
//
// All code is compiled with -ffp-contract=off; fused multiply-adds are
// written explicitly where wanted, and the scalar move arithmetic keeps the
// operation order of its definition.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <map>
#include <thread>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <string>
#include <vector>

#include "sail.h"

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr uint32_t kStreamProposal = 0u;
constexpr uint32_t kStreamBranch = 0x42524E43u;
constexpr int kThreads = 256;
constexpr int kBranchThreads = 1024;
constexpr int kBranchWPT = 16;  // walkers per thread in the branching solve
constexpr int kBranchMaxWalkers = kBranchThreads * kBranchWPT;
constexpr int kMaxWalk = 64;  // longest index-selection walk

thread_local std::string g_err;

sail_status fail(sail_status s, const std::string &msg)
{
    g_err = msg;
    return s;
}

#define SAIL_HIP(call)                                                                        \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return fail(SAIL_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

// --------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11)
// --------------------------------------------------------------------------
__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                         uint32_t k1, uint32_t &o0, uint32_t &o1, uint32_t &o2, uint32_t &o3)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // the 64-bit products give both halves in one multiply-add each
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        // three-input XOR in one instruction (truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    o0 = c0;
    o1 = c1;
    o2 = c2;
    o3 = c3;
}

// word -> open unit interval, (x + 1/2) 2^-32 = x 2^-32 + 2^-33 (exact either
// way for a 32-bit x, so one FMA gives the same bits); word -> index, high
// half of x*n
__device__ __forceinline__ double u01(uint32_t x)
{
    return fma((double)x, 2.3283064365386962890625e-10, 1.16415321826934814453125e-10);
}
__device__ __forceinline__ int index_of(uint32_t x, int n) { return (int)__umulhi(x, (uint32_t)n); }

// 1/x from the FP32 reciprocal and two Newton steps: a few units in the last
// place for the operands used here (bin spacings and r in [1 - eps0, 1 + eps0]).
__device__ __forceinline__ double recip(double x)
{
    double y = (double)__builtin_amdgcn_rcpf((float)x);
    y = fma(y, fma(-x, y, 1.0), y);
    y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// The two deltas of Eqs. (update-delta-p/s) with bin centres, through one
// shared reciprocal of w_p - w_s (the sums they preserve hold to rounding).
__device__ __forceinline__ void move_deltas(double A, double B, double wp, double ws, double r, double &dp, double &ds)
{
    const double inv = recip(wp - ws), omr = 1.0 - r;
    dp = omr * (B - A * ws) * inv;
    ds = -(omr * (B - A * wp) * inv);
}

// Staged accept threshold: -T ln u from the FP32 log2.  With u rounded to
// FP32 (relative 2^-24, so ln u moves by <= 6e-8) and log2 good to a few FP32
// units in the last place (relative <= 5e-7 of |log2 u| <= 33), the staged
// value lies within kThrTol (|thr| + T) of the exact -T ln u; a decision
// closer than that to the staged threshold is retaken with the exact one.
constexpr double kLn2 = 0.69314718055994530941723212145818;
constexpr double kThrTol = 4e-6;
__device__ __forceinline__ double staged_threshold(double T, double u)
{
    return -T * ((double)__builtin_amdgcn_logf((float)u) * kLn2);
}

// --------------------------------------------------------------------------
// Sweep kernel: sweeps [k0, k1) for every walker (Sec. 2.2, 2.3, 2.7).
// --------------------------------------------------------------------------
struct SweepArgs {
    int n_walkers, n_omega;
    int k0, k1;
    uint32_t key0, key1;
    double A, B, eps0, amp_p, amp_avg;
    int amp_m;
    int columns_lds;      // 1: the workgroup copies the columns to LDS
    int tables_lds;       // columns in memory: it copies the table values of bins (1), of bins and pairs (2)
    int resident;         // split sweeps: bins of every spectrum, the first ones, that the workgroup keeps in LDS
    int lanes;            // lanes a walker takes (a batch's split sweeps: 4 or 16)
    int pairs;            // split sweeps: chain and stager wavefronts at work in a workgroup (any others leave)
    const void *col;      // [N_omega][4][chunk] columns in the basis, loop precision
    void *phi;            // [N_w][4][chunk] walkers in the basis, loop precision
    // the parts of the residue change that do not depend on the walker (FP64):
    // D_j = sum_i w_i K_ij^2, V_j = sum_i c_i K_ij with c_i = -2 w_i Phit_i, and
    // (G_k, H_k) = sum_i w_i (1, tau_i) e^{-wbar_k tau_i} on the pair sums
    // wbar_k = 2 omega_0 + k d_omega, with C = sum_i w_i Phit_i^2
    const double4 *bin;   // [N_omega] (omega_j, D_j, V_j, 0)
    const double2 *GH;    // [2 N_omega - 1]
    double C, w0, dW;
    double *b;            // [N_w][N_omega] spectra up to the lazy scale
    double *gsc, *ginv, *chi2, *rate;  // [N_w]; ginv carries 1/g as the product of the moves' 1/r
    const double *Tabs;   // [n_T] absolute temperature of each global sweep
    int tk0, tk1;         // trace window
    double *tr_dchi2;
    uint8_t *tr_flags;
    int wg_sync;          // 1: workgroup barrier between record staging and use (diagnostic)
    int walk_len;         // steps of the index-selection walk (Sec. 2.3); 0: uniform p, s
    double thr_tol;       // relative band of the staged threshold (infinite: always the FP64 log; diagnostic)
};

// Butterfly sum over the L lanes of a walker with DPP lane swaps (rows of
// 16 lanes); every lane ends with the same bits because each step adds two
// equal-shaped partial sums in commutative order.
template <int CTRL>
__device__ __forceinline__ double dpp_swap(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Lane t (a compile-time number) of the walker's G = 4 or 16 lanes, by DPP
// (quad_perm, row_newbcast).
template <int G>
__device__ __forceinline__ int lane_of(const int x, const int t)
{
#define SAIL_LANE(n, ctrl) case n: return __builtin_amdgcn_mov_dpp(x, ctrl, 0xF, 0xF, true);
    if constexpr (G == 4) {
        switch (t) {
            SAIL_LANE(0, 0x00) SAIL_LANE(1, 0x55) SAIL_LANE(2, 0xAA)
            default: return __builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, true);
        }
    } else {
        static_assert(G == 16, "a quad or a row");
        switch (t) {
            SAIL_LANE(0, 0x150) SAIL_LANE(1, 0x151) SAIL_LANE(2, 0x152) SAIL_LANE(3, 0x153) SAIL_LANE(4, 0x154)
            SAIL_LANE(5, 0x155) SAIL_LANE(6, 0x156) SAIL_LANE(7, 0x157) SAIL_LANE(8, 0x158) SAIL_LANE(9, 0x159)
            SAIL_LANE(10, 0x15A) SAIL_LANE(11, 0x15B) SAIL_LANE(12, 0x15C) SAIL_LANE(13, 0x15D) SAIL_LANE(14, 0x15E)
            default: return __builtin_amdgcn_mov_dpp(x, 0x15F, 0xF, 0xF, true);
        }
    }
#undef SAIL_LANE
}

template <int CTRL>
__device__ __forceinline__ float dpp_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ int dpp_swap(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}

template <int L, typename R>
__device__ __forceinline__ R group_sum(R v)
{
    if (L >= 2) v = v + dpp_swap<0xB1>(v);   // quad_perm [1,0,3,2]: lane ^ 1
    if (L >= 4) v = v + dpp_swap<0x4E>(v);   // quad_perm [2,3,0,1]: lane ^ 2
    if (L >= 8) v = v + dpp_swap<0x141>(v);  // row_half_mirror: quads of an 8-lane half
    if (L >= 16) v = v + dpp_swap<0x140>(v); // row_mirror: halves of a 16-lane row
    if (L >= 32) v = v + __shfl_xor(v, 16, 64);
    if (L >= 64) v = v + __shfl_xor(v, 32, 64);
    return v;
}

// Orders a wavefront's LDS writes before its later LDS reads by other lanes.
// A wavefront's LDS operations are performed in order, so this only has to
// stop the compiler from moving memory operations across it.
__device__ __forceinline__ void wave_lds_sync()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Per-proposal quantities that do not depend on the walker state, computed
// for a batch of G proposals at once (lane c of a walker takes proposal
// q0 + c) and staged in LDS, read in 16-byte pairs: r - 1, 1/r, the accept
// threshold, the walker-independent parts of the residue change, S1 =
// sum_i w_i s_i^2 and S1 + S3 with S3 = sum_i c_i s_i (s_i = dp K_pi + ds K_si),
// the deltas dp and ds, and the bins, each twice in one word (p | p << 16,
// s | s << 16), or the threshold's band.  The bins also stand apart: they are
// read a proposal earlier than the rest.
enum : int {
    kRecRm1 = 0, kRecRinv = 1, kRecThr = 2, kRecT = 3, kRecS1 = 4, kRecDp = 5, kRecDs = 6, kRecPS = 7,
    kRecBand = 7  // split sweeps, which stage masks of shared bins instead: the threshold's band
};
constexpr int kRecWords = 8;      // doubles per record
constexpr int kWalkWords = 5;     // doubles per staged step of an index-selection walk: bins, two values, two draws
// Threshold of a proposal that is never accepted: nothing compares below it, a
// residue change of -infinity (an infinite residue's) included, or near it.
constexpr double kNever = __builtin_nan("");
// Doubles of LDS per walker, padded against bank conflicts: the records and
// bins of two batches (one runs while the next is staged), or of one batch and
// its walk steps.
constexpr int rec_stride(int G, bool walk) { return (walk ? G * (kRecWords + 1 + kWalkWords) : 2 * G * (kRecWords + 1)) + 2; }

// A split sweep's walker: records of three batches, bins of four, the move
// width; and a wavefront's masks of shared bins of three batches.
constexpr int split_hits(int G) { return 3 * G; }
constexpr int split_stride(int G) { return 3 * G * kRecWords + 4 * G + 2; }

// A split walk's walker: of two batches of 16 proposals, the records (r - 1 or
// its draw, 1/r, the threshold and the uniform bins) and the walk's steps (two
// words a side: the candidate bin and its draw); the move width.
constexpr int kWalkRec = 4;
constexpr int64_t walk_split_stride(int walk_len) { return (int64_t)2 * 16 * (kWalkRec + (int64_t)2 * walk_len) + 2; }

// Basis dimensions per chunk as stored: whole 16-byte words.
template <typename R>
constexpr int chunk_stride(int m) { return sizeof(R) == 8 ? (m + 1) & ~1 : (m + 3) & ~3; }

// The sweep kernels are built for these numbers of dimensions per chunk.  Decaying
// kernels take up to 8; weights that turn the columns into separate Gaussians
// more, which are held by 16 lanes, a quarter of a chunk each (96 bins, 96 x 4
// dimensions at most, 1024 walkers: 235 ns a proposal, 3.3 us with a walker's
// coordinates in memory, 470 ns with a recurrence along 80 times).  More than 4096
// walkers leave a compute unit 16 at a time and stay behind the recurrence (8192: 760
// against 540 us for 960 proposals).  The widest (500 bins, 512 times, 1024 walkers, FP64):
// four sweeps 0.98 ms, 15.8 with the coordinates in memory, 1.31 with the recurrence.
constexpr int kDims64[7] = {2, 4, 6, 8, 16, 24, 32}, kDims32[6] = {2, 3, 4, 6, 16, 24};
constexpr int kBasisClasses = 33;
constexpr bool wide_basis(int m) { return m > 8; }
constexpr int kReadRows = 16;  // walkers whose reconstructions are read at once, at least
// Dimensions per chunk for a basis of n dimensions (or the most there are).
int round_dims(int precision, int n)
{
    const int need = n > 4 ? (n + 3) / 4 : 1;
    const int *m = precision == SAIL_FP32 ? kDims32 : kDims64, *last = m + (precision == SAIL_FP32 ? 5 : 6);
    while (m < last && need > *m) ++m;
    return *m;
}

size_t column_bytes(int n_omega, int chunk, size_t rsz) { return (size_t)n_omega * 4 * chunk * rsz; }

// Workgroups go to the XCDs in turn; within a window of kXcdWindow of them (one a
// compute unit), give each XCD neighbouring ones, so that the tables of few
// problems share its L2 cache: for launches that read columns from memory (32 jobs of
// 2000 bins, 2000 walkers: 16.5 to 10.4 ms).  Where the columns are in LDS the caches
// hold spectra, and the largest jobs' would all meet in one (16 served FP32 jobs:
// 20.8 to 24.4 ms).
constexpr int kXcds = 8, kXcdWindow = 256;
__device__ __forceinline__ int xcd_block(const int b, const int n)
{
    const int base = b / kXcdWindow * kXcdWindow, m = min(n - base, kXcdWindow), x = (b - base) % kXcds, i = (b - base) / kXcds;
    return base + x * (m / kXcds) + min(x, m % kXcds) + i;
}

// Many problems in one launch: problem q owns workgroups [first[q], first[q + 1]).
__device__ __forceinline__ int owner_of(const int *first, const int n_jobs, const int b)
{
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Raw buffer access with 32-bit byte offsets (gfx9 resource word 3 = 0x00020000);
// offsets past `bytes` read as zero and drop stores.
constexpr uint32_t kDropStore = 0x80000000u;  // past every buffer the kernels address (< 2 GiB)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ double buffer_load_f64(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    double d;
    __builtin_memcpy(&d, &v, sizeof d);
    return d;
}

__device__ __forceinline__ void buffer_store_f64(__amdgpu_buffer_rsrc_t r, uint32_t off, double d)
{
    decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)) v;
    __builtin_memcpy(&v, &d, sizeof d);
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
}

// One lane's chunk of a column: M values in 16-byte loads.  From memory, the last
// one takes the values that are left: a full one would let its unused registers
// overlap another load's, which then waits for it (FP32, 2556 bins x 5000 walkers: 455 to
// 285 ns a proposal).  From LDS full ones are faster (ds_read_b96, FP32, 300 bins x
// 3000 walkers: 211 to 229 ns).  Quarters of a chunk that end within 16 bytes (FP32, 24
// dimensions a chunk) are loaded by 8.
template <bool MEM, typename R, int M, int BYTES = 16>
__device__ __forceinline__ void load_chunk(const R *p, R (&v)[M])
{
    constexpr int W = BYTES / sizeof(R), MS = (M + W - 1) / W * W;
    typedef R vec __attribute__((ext_vector_type(W)));
    typedef R pair __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < MS; i += W) {
        if (!MEM || i + W <= M) {
            const vec x = *(const vec *)(p + i);
#pragma unroll
            for (int t = 0; t < W; ++t)
                if (i + t < M) v[i + t] = x[t];
        } else {
            const R *q = (const R *)__builtin_assume_aligned(p + i, 16);
            if (M - i >= 2) {
                const pair x = *(const pair *)q;
                v[i] = x[0];
                v[i + 1] = x[1];
            }
            if ((M - i) % 2) v[M - 1] = q[M - 1 - i];
        }
    }
}

// Lanes qq, qq + G, qq + 2 G, ...: the owners of proposal qq of a batch.
template <int G>
__device__ __forceinline__ uint64_t owner_lanes(int qq)
{
    constexpr uint64_t base = G == 4 ? 0x1111111111111111ull : G == 8 ? 0x0101010101010101ull : 0x0001000100010001ull;
    static_assert(G == 4 || G == 8 || G == 16, "lanes per walker");
    return base << qq;
}

// What a launch of the sweep does: uniform selection; the same with the
// per-proposal trace; index selection by walks (with the trace, if it is on).
enum : int { kSweepFast = 0, kSweepTraced = 1, kSweepWalk = 2 };

// The sweep of one workgroup's walkers: `block` numbers the workgroup within
// the problem, `lds` is its LDS (records, then the columns if LDSC, then the
// walkers' spectra if LDSB).  R is the precision of the residual loop (double:
// the FP64 path, float: the FP32 variant); moves, positivity, thresholds and
// chi^2 stay double.  M is the number of basis dimensions a chunk holds; a wide
// basis (more than 8) takes 16 lanes, each with a quarter of a chunk.
//
// SPLIT: half of the workgroup's wavefronts run the walkers' chains, four lanes
// a walker; the other half, one beside each on the same SIMD, draw and stage
// the proposals for them.  A chain's proposal is a serial sequence of some
// hundred instructions, mostly waiting on its own results, so the staging's
// instructions cost little beside it and a lot within it (512 bins, four lanes,
// spectra in memory: 1024 walkers 378 ns a proposal in one wavefront and 250 ns
// split, 16384 walkers 441 and 393 ns).
template <typename R, int M, int G, bool LDSC, bool LDSB, int MODE, bool SPLIT>
__device__ __forceinline__ void sweep_block(const SweepArgs &a, const int block, double *lds)
{
    constexpr bool WALK = MODE == kSweepWalk, TRACE = MODE != kSweepFast;
    constexpr bool WIDE = wide_basis(M);
    constexpr int CH = WIDE ? 16 : 4, MR = 4 * M / CH;  // lanes that share a walker's coordinates, dimensions in each
    static_assert(!WIDE || G == 16, "a wide basis takes 16 lanes");
    const int RSTR = !SPLIT ? rec_stride(G, WALK) : WALK ? (int)walk_split_stride(a.walk_len) : split_stride(G);
    static_assert(!SPLIT || (WALK ? G == 16 && LDSB : G == 16 || G == 4), "split sweeps");
    constexpr bool ALLB = LDSB && (!SPLIT || G == 16);  // whole spectra in LDS; split sweeps keep the first bins there
    const int nthr = SPLIT ? 128 * a.pairs : (int)blockDim.x;
    if (SPLIT && (int)threadIdx.x >= nthr) return;
    const int lane = threadIdx.x & 63;
    const int c = lane & (G - 1), ch = lane & (CH - 1);
    // walkers of the workgroup, and this lane's among them
    const int half = nthr >> 1;
    const bool stager = SPLIT && (int)threadIdx.x >= half;
    const int wpb = (SPLIT ? half : nthr) / G, ws = (int)(stager ? threadIdx.x - half : threadIdx.x) / G;
    const int l = block * wpb + ws;
    const bool valid = l < a.n_walkers;
    const int lw = valid ? l : a.n_walkers - 1;
    const int No = a.n_omega;
    // descriptor fields the loops use, read once: the batched kernel reads its
    // descriptor from global memory, which the loops' stores might alias, so
    // every use inside a loop would be a fresh load and wait
    const uint32_t key0 = a.key0, key1 = a.key1;
    const double Asum = a.A, Bsum = a.B, thr_tol = a.thr_tol;
    const double amp_p = a.amp_p, amp_avg = a.amp_avg, eps0 = a.eps0;
    const int amp_m = a.amp_m, walk_len = a.walk_len, wg_sync = a.wg_sync, k1 = a.k1;
    const double *Tsched = a.Tabs;
    const double4 *bin = a.bin;
    const double2 *GH = a.GH;
    const double cC = a.C, w0x2 = 2.0 * a.w0, dW = a.dW;
    constexpr int st = WIDE ? MR : chunk_stride<R>(MR), CVAL = CH * st;  // stored dimensions: of a lane, of a column
    constexpr int LB = st * sizeof(R) % 16 ? 8 : 16;                     // bytes of a load
    const int mine = WIDE ? (ch & 3) * (4 * st) + (ch >> 2) * st : ch * st;  // where this lane's are

    // records, columns and spectra in LDS
    double *myrec = lds + ws * RSTR;
    const R *colg = (const R *)a.col;
    R *col_s = (R *)(lds + wpb * RSTR + (SPLIT && !ALLB ? wpb / (64 / G) * split_hits(G) : 0));
    if constexpr (LDSC) {
        const size_t n16 = (size_t)No * CVAL * sizeof(R) / 16;
        for (size_t i = threadIdx.x; i < n16; i += nthr) ((float4 *)col_s)[i] = ((const float4 *)colg)[i];
    }
    double *spec = (double *)(col_s + (LDSC ? (size_t)No * CVAL : 0));
    // the walker's spectrum, or its first bins and a slot for the others' stores
    const int nres = ALLB ? No : a.resident;
    double *bsp = spec + (size_t)ws * (ALLB ? No : nres + 1);
    if constexpr (LDSB) {
        const double *bl = a.b + (size_t)lw * No;
        for (int j = c; j < nres && !stager; j += G) bsp[j] = bl[j];
    }
    // Table values of bins and pairs in LDS: of a split walk, whose bins are known
    // late, and where the columns are in memory (a batch of problems' columns and
    // tables would not stay in the caches; 32 jobs of 2556 bins, 300 walkers: with
    // all table reads to one place a launch takes 3.36 instead of 4.42 ms)
    constexpr bool TAB = (SPLIT && WALK) || !LDSC;
    const bool bins_in = (SPLIT && WALK) || (TAB && a.tables_lds > 0), pairs_in = (SPLIT && WALK) || (TAB && a.tables_lds > 1);
    double4 *bin_s = (double4 *)(spec + (LDSC ? ((size_t)wpb * No + 1) & ~(size_t)1 : 0));
    double2 *GH_s = (double2 *)(bin_s + No);
    if (bins_in)
        for (int i = threadIdx.x; i < No; i += nthr) bin_s[i] = bin[i];
    if (pairs_in)
        for (int i = threadIdx.x; i < 2 * No - 1; i += nthr) GH_s[i] = GH[i];
    __syncthreads();

    // spectra in memory through a buffer resource: 32-bit offsets (the library
    // keeps the array below 2 GiB)
    const __amdgpu_buffer_rsrc_t b_rs = buffer_of(a.b, (uint32_t)((size_t)a.n_walkers * No * sizeof(double)));
    const uint32_t brow = (uint32_t)((size_t)lw * No * sizeof(double));  // byte offset of the walker's spectrum
    auto load_b = [&](const int j) __attribute__((always_inline)) {
        if constexpr (ALLB) return bsp[j];
        else return buffer_load_f64(b_rs, brow + ((uint32_t)j << 3));
    };

    R phi[MR], lost = 0;  // lost: FP32, of a sweep's additions to phi[0]
    R *phig = (R *)a.phi + (size_t)lw * CVAL + mine;
    load_chunk<false, R, MR, LB>(phig, phi);
    double g = a.gsc[lw], chi2 = a.chi2[lw], rate = a.rate[lw], ginv = a.ginv[lw];
    double Q2 = 0.0;  // sum_i w_i Phi_i^2 of the walker, from its coordinates at each sweep's start
    int nacc = 0;
    int k = a.k0, q0 = 0;
    double Tabs = 0.0, yeps = 0.0, thr_T = 0.0;  // temperature and move width of sweep k, thr_tol T

    // Spectra in memory: the proposal this lane owns in the current batch (its
    // bins' spectrum values here, stored when the batch has ended) and in the
    // next one, whose values load while the current batch runs; values that
    // an accepted move of the current batch replaces wait beside them.
    int op = 0, os = 0, np_ = 0, ns_ = 0;
    uint32_t ops = 0, nps = 0, nx2 = 0, nx3 = 0;
    double obp = 0.0, obs = 0.0, nbp = 0.0, nbs = 0.0, fbp = 0.0, fbs = 0.0;
    uint32_t fp = 0, fs = 0;  // not 0: fbp, fbs replace nbp, nbs (words, not lane masks: they change in few lanes, rarely)
    uint64_t accm = 0;        // owner lanes whose proposal of the current batch was accepted
    const uint64_t validm = __builtin_amdgcn_ballot_w64(valid);
    int buf = 0;              // half of the staging area the current batch reads

    struct Rec {
        int p, s;
        uint32_t pp, ss;  // p | p << 16, s | s << 16
        double rm1, rinv, thr, t, s1, dp, ds, band;
        R rp[MR], rs[MR];
    };

    auto rows = [&](int p, int s, Rec &v) __attribute__((always_inline)) {
        // (keeps the halves apart: shifts of the whole word cost more)
        asm("" : "+v"(p), "+v"(s));
        v.p = p;
        v.s = s;
        const uint32_t po = (uint32_t)p * CVAL + (uint32_t)mine, so = (uint32_t)s * CVAL + (uint32_t)mine;
        if constexpr (LDSC) {
            load_chunk<false, R, MR, LB>(col_s + po, v.rp);
            load_chunk<false, R, MR, LB>(col_s + so, v.rs);
        } else {
            load_chunk<true, R, MR, LB>(colg + po, v.rp);
            load_chunk<true, R, MR, LB>(colg + so, v.rs);
        }
    };
    // staging area of a walker: records of batch slot h, then the bins
    auto rec_at = [&](const int h, const int qq) __attribute__((always_inline)) { return myrec + (h * G + qq) * kRecWords; };
    auto bins_at = [&](const int h, const int qq) __attribute__((always_inline)) {
        return myrec + (SPLIT ? 3 : WALK ? 1 : 2) * G * kRecWords + h * G + qq;
    };
    auto fetch = [&](const double *rc, Rec &v) __attribute__((always_inline)) {
        v.rm1 = rc[kRecRm1];
        v.rinv = rc[kRecRinv];
        v.thr = rc[kRecThr];
        v.t = rc[kRecT];
        v.s1 = rc[kRecS1];
        v.dp = rc[kRecDp];
        v.ds = rc[kRecDs];
        const double w = rc[kRecPS];
        if constexpr (SPLIT) {
            v.band = w;
        } else {
            v.pp = (uint32_t)__double2loint(w);
            v.ss = (uint32_t)__double2hiint(w);
        }
    };

    // Table values of a pair of bins: loaded a batch ahead, so that staging a
    // record waits for no memory.
    struct Pair {
        double4 p, s;
        double2 gh;
    };
    auto load_pair = [&](const int p, const int s, Pair &t) __attribute__((always_inline)) {
        if (TAB && bins_in) {
            t.p = bin_s[p];
            t.s = bin_s[s];
        } else {
            t.p = bin[p];
            t.s = bin[s];
        }
        if (TAB && pairs_in) t.gh = GH_s[p + s];
        else t.gh = GH[p + s];
    };
    // Deltas and walker-independent residue terms of the move (p, s, r): S1 =
    // sum_i w_i s_i^2 and S1 + S3 (S3 = sum_i c_i s_i); sum_i w_i K_pi K_si is
    // the pair-sum entry G at wbar = 2 omega_0 + (p + s) d_omega, moved to
    // omega_p + omega_s to first order by H (the grid is uniform to rounding,
    // so the shift is tiny).  p = s moves nothing.
    auto pair_terms = [&](const int p, const int s, const Pair &t, const double r, double &dp, double &ds, double &s1_,
                          double &t_) __attribute__((always_inline)) {
        move_deltas(Asum, Bsum, t.p.x, t.s.x, r, dp, ds);
        dp = p == s ? 0.0 : dp;
        ds = p == s ? 0.0 : ds;
        const double shift = (t.p.x + t.s.x) - (w0x2 + (double)(p + s) * dW);
        const double mps = t.gh.x - shift * t.gh.y;
        const double S1 = dp * dp * t.p.y + 2.0 * dp * ds * mps + ds * ds * t.s.y;
        s1_ = S1;
        t_ = S1 + (dp * t.p.z + ds * t.s.z);
    };

    // the uniform draws of proposal q of sweep kk
    auto draw = [&](const int q, const int kk, int &p, int &s, uint32_t &x2, uint32_t &x3)
                    __attribute__((always_inline)) {
        uint32_t x0, x1;
        philox10((uint32_t)q, (uint32_t)kk, (uint32_t)lw, kStreamProposal, key0, key1, x0, x1, x2, x3);
        p = index_of(x0, No);
        s = index_of(x1, No);
    };

    // writes the bins of this lane's proposal q of a batch (past N_omega: 0, 0)
    auto stage_bins = [&](const int h, const int q, const int p, const int s) __attribute__((always_inline)) {
        const bool in = q < No;
        *bins_at(h, c) = __hiloint2double(in ? s : 0, in ? p : 0);
    };
    // writes its record.  Past N_omega the record is a no-op: r = 1, never
    // accepted.  Straight-line code: it runs in the latencies of the batch
    // before.
    auto stage = [&](const int h, const int q, const int p, const int s, const uint32_t x2, const uint32_t x3,
                     const Pair &pr) __attribute__((always_inline)) {
        double *rcw = rec_at(h, c);
        const bool in = q < No;
        const double ur = u01(x2), ua = u01(x3);
        // r from the rounded r - 1 (exact for r in [1/2, 2]): both are used
        const double rm1 = in ? (1.0 - yeps * fma(2.0, ur, -1.0)) - 1.0 : 0.0;  // 2u - 1 is exact either way
        const double r = rm1 + 1.0;
        double s1t = 0.0, tt = 0.0, dp = 0.0, ds = 0.0;
        if constexpr (!WALK) pair_terms(p, s, pr, r, dp, ds, s1t, tt);
        // u < e^{-dchi2/T}  <=>  dchi2 < -T ln u  (T > 0); p = s is never
        // accepted
        const double thr = staged_threshold(Tabs, ua);
        rcw[kRecRm1] = rm1;
        rcw[kRecRinv] = recip(r);
        rcw[kRecThr] = (!in | (!WALK && p == s)) ? kNever : thr;
        rcw[kRecT] = tt;
        rcw[kRecS1] = s1t;
        rcw[kRecDp] = dp;
        rcw[kRecDs] = ds;
        if constexpr (SPLIT) rcw[kRecBand] = fma(fabs(rcw[kRecThr]), thr_tol, thr_T);
        else rcw[kRecPS] = __hiloint2double((in ? s : 0) * 0x10001, (in ? p : 0) * 0x10001);
    };

    // Lanes where a half of w is zero, and the smaller of two words by halves.
    auto zero_half = [&](const uint32_t w) __attribute__((always_inline)) {
        return __builtin_amdgcn_ballot_w64((w & 0xffffu) == 0u) | __builtin_amdgcn_ballot_w64(w < 0x10000u);
    };
    typedef unsigned short half2 __attribute__((ext_vector_type(2)));
    auto min_halves = [&](const uint32_t x, const uint32_t y) __attribute__((always_inline)) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(half2, x), __builtin_bit_cast(half2, y)));
    };

    // lanes holding a bin of proposal qq (packed pp, ss) for another proposal of
    // its batch (ops) or for the next batch (nps)
    auto shared_bins = [&](const int qq, const uint32_t pp, const uint32_t ss) __attribute__((always_inline)) {
        const uint32_t hc = min_halves(ops ^ pp, ops ^ ss), hn = min_halves(nps ^ pp, nps ^ ss);
        return zero_half(min_halves(__builtin_amdgcn_inverse_ballot_w64(owner_lanes<G>(qq)) ? 0xffffffffu : hc, hn));
    };
    // the value lane lead + qq of the walker holds
    auto of_owner = [&](const double x, const int qq) __attribute__((always_inline)) {
        if constexpr (SPLIT || G == 4) return __hiloint2double(lane_of<G>(__double2hiint(x), qq), lane_of<G>(__double2loint(x), qq));
        else return __shfl(x, (lane & ~(G - 1)) + qq, 64);
    };

    // One proposal: v is its record and columns, bp and bs the spectrum values
    // of its bins: in every lane of the walker, or, with spectra in memory and
    // uniform selection, in its owner lanes.
    // hit: with staged masks (SPLIT), the lanes of walkers with a bin of this
    // proposal elsewhere in the batch or in the next one.
    auto body = [&](const int qq, const Rec &v, const double bp, const double bs, const uint64_t hit)
                    __attribute__((always_inline)) {
        constexpr bool OWNED = !WALK && !ALLB;
        const double rm1d = v.rm1, r = v.rm1 + 1.0;
        // F' = r F + s with s_i = dp K_pi + ds K_si.  The residue change
        // sum_i w_i ((Phi'_i - Phit_i)^2 - (Phi_i - Phit_i)^2) expands into
        //   (r - 1) (r Q2 + chi^2 - C) + 2 r S2 + S1 + S3,
        // Q2 = sum_i w_i Phi_i^2 (the walker's, from its coordinates at each sweep's
        // start, short of it by what the basis leaves of Phi, squared, and
        // carried through the accepted moves), S2 = sum_i w_i Phi_i s_i =
        // phi . sigma (the only sum that needs the walker), and S1 =
        // sum_i w_i s_i^2, S3 = sum_i c_i s_i from tables (staged);
        // chi^2 - Q2 - C = sum_i c_i Phi_i.  Every term is bounded by the
        // condition scale of the direct sum, so the expansion keeps its
        // rounding error (with r^2 - 1 taken as (r - 1)(r + 1), r - 1 exact).
        // The part of s outside the basis meets the part of Phi outside it
        // only: the two residuals' product is what the basis leaves out.
        R sv[MR], acc = 0;
        const R dpr = (R)v.dp, dsr = (R)v.ds;
#pragma unroll
        for (int t = 0; t < MR; ++t) {
            sv[t] = fma(dpr, v.rp[t], dsr * v.rs[t]);
            acc = t == 0 ? phi[t] * sv[t] : fma(phi[t], sv[t], acc);
        }
        const double S2 = (double)group_sum<CH>(acc);
        const double r2 = r + r;
        const double dchi2 = fma(rm1d, fma(r, Q2, chi2 - cC), fma(r2, S2, v.t));
        // r g, exactly rounded (r - 1 is exact, so g (r - 1) + g is g r): the
        // scale after an accepted move and the factor of the positivity test
        const double rg = fma(rm1d, g, g);
        const double ap = fma(rg, bp, v.dp), as = fma(rg, bs, v.ds);
        const double diff = dchi2 - v.thr;
        // (decisions are lane masks, combined by the scalar unit, which also
        // spreads the owner lane's positivity over the walker's G lanes)
        const uint64_t own = owner_lanes<G>(qq);
        uint64_t pos = __builtin_amdgcn_ballot_w64(ap >= 0.0) & __builtin_amdgcn_ballot_w64(as >= 0.0);
        if constexpr (OWNED) {
            const uint64_t bit = (pos & own) >> qq;
            pos = (bit << G) - bit;
        }
        if constexpr (WALK) pos &= __builtin_amdgcn_ballot_w64(v.p != v.s);
        uint64_t am = pos & __builtin_amdgcn_ballot_w64(diff < 0.0);
        // a decision within thr_tol (|thr| + T) of the staged threshold is
        // retaken with the exact logarithm
        const uint64_t near = pos & __builtin_amdgcn_ballot_w64(fabs(diff) <= (SPLIT && !WALK ? v.band : fma(fabs(v.thr), thr_tol, thr_T)));
        if (__builtin_expect(near != 0, 0)) {  // (out of line: a taken branch costs the common path)
            bool take = false;
            if (__builtin_amdgcn_inverse_ballot_w64(near)) {
                uint32_t x0, x1, x2, x3;
                philox10((uint32_t)(q0 + qq), (uint32_t)k, (uint32_t)lw, kStreamProposal, key0, key1, x0, x1, x2, x3);
                take = dchi2 < -Tabs * log(u01(x3));
            }
            am = (am & ~near) | (near & __builtin_amdgcn_ballot_w64(take));
        }
        if (TRACE && k >= a.tk0 && k < a.tk1) {
            if (c == qq && valid && q0 + qq < No) {
                const size_t o = ((size_t)l * (size_t)(a.tk1 - a.tk0) + (size_t)(k - a.tk0)) * No + q0 + qq;
                a.tr_dchi2[o] = dchi2;
                a.tr_flags[o] = (uint8_t)((__builtin_amdgcn_inverse_ballot_w64(am) ? 1 : 0) |
                                          (__builtin_amdgcn_inverse_ballot_w64(pos) && v.p != v.s ? 2 : 0));
            }
        }
        if constexpr (OWNED) accm |= am & own;
        if (__builtin_amdgcn_inverse_ballot_w64(am)) {
            if constexpr (sizeof(R) == 8) {
                // the three-operand FMA writes phi in place (the compiler's
                // accumulating form lands in sv and needs a copy back each)
#pragma unroll
                for (int t = 0; t < MR; ++t) asm("v_fma_f64 %0, %1, %0, %2" : "+v"(phi[t]) : "v"(r), "v"(sv[t]));
            } else {
                // FP32: r - 1 rounds to FP32 with a relative error far smaller
                // than r would, so the change is formed first.  What an addition to a
                // lane's first value, the largest by far (the basis is in principal
                // directions), loses is carried to the next one until the sweep ends:
                // without, residue changes fifty sweeps after a resync were off by
                // 8.6e-8 of their condition scale (rms, 512 bins x 128 times), with it
                // by 1.5e-8, and by 3.7e-8 with FP32 values per time, whose roundings
                // averaged (512 bins x 16384 walkers, block 18.3 to 18.6 ms)
                const R rm1 = (R)rm1d;
#pragma unroll
                for (int t = 0; t < MR; ++t) {
                    const R y = fma(rm1, phi[t], t == 0 ? sv[t] + lost : sv[t]), sum = phi[t] + y;
                    if (t == 0) lost = y - (sum - phi[t]);
                    phi[t] = sum;
                }
            }
            asm("v_fma_f64 %0, %1, %0, %2" : "+v"(Q2) : "v"(r * r), "v"(fma(r2, S2, v.s1)));
            chi2 = chi2 + dchi2;
            g = rg;
            ginv = ginv * v.rinv;
            ++nacc;
            // the pair's new spectrum values, scaled by the new 1/g
            const double bpn = ap * ginv, bsn = as * ginv;
            if constexpr (ALLB) {
                if (c == 0) {
                    bsp[v.p] = bpn;
                    bsp[v.s] = bsn;
                }
            } else if constexpr (WALK) {
                // the next walk reads the spectrum: store at once
                if (valid && c == 0) {
                    buffer_store_f64(b_rs, brow + ((uint32_t)v.p << 3), bpn);
                    buffer_store_f64(b_rs, brow + ((uint32_t)v.s << 3), bsn);
                }
            } else {
                // they stay with their owner until the batch ends; any lane that
                // holds one of the two bins, for this batch or the next, takes
                // them over (few walkers per proposal: a branch on the whole
                // wavefront; the next batch's values, still in flight, are not
                // touched)
                if (__builtin_amdgcn_inverse_ballot_w64(own)) {
                    obp = bpn;
                    obs = bsn;
                }
                if (am & (SPLIT ? hit : shared_bins(qq, v.pp, v.ss))) {
                    const double vp = of_owner(bpn, qq), vs = of_owner(bsn, qq);
                    if (__builtin_amdgcn_inverse_ballot_w64(~own)) {
                        obp = op == v.p ? vp : op == v.s ? vs : obp;
                        obs = os == v.p ? vp : os == v.s ? vs : obs;
                    }
                    fbp = np_ == v.p ? vp : np_ == v.s ? vs : fbp;
                    fbs = ns_ == v.p ? vp : ns_ == v.s ? vs : fbs;
                    fp = ((np_ == v.p) | (np_ == v.s)) ? 1u : fp;
                    fs = ((ns_ == v.p) | (ns_ == v.s)) ? 1u : fs;
                    asm volatile("" : "+v"(fp), "+v"(fs));
                }
            }
        }
    };

    // starts sweep k: temperature, amplitude (Eq. amplitude-acceptance-adjustment
    // on the running acceptance rate) and the exact Q2
    auto temperature = [&]() __attribute__((always_inline)) {
        Tabs = Tsched[k];
        thr_T = thr_tol * Tabs;
    };
    auto begin_sweep = [&]() __attribute__((always_inline)) {
        temperature();
        double y = 1.0;
        if (rate < amp_p) {
            const double q = rate / amp_p;
            for (int m = 0; m < amp_m; ++m) y = y * q;
        }
        yeps = y * eps0;
        nacc = 0;
        double q2 = 0.0;
#pragma unroll
        for (int t = 0; t < MR; ++t) q2 = fma((double)phi[t], (double)phi[t], q2);
        lost = 0;
        Q2 = group_sum<CH>(q2);
    };
    auto end_sweep = [&]() __attribute__((always_inline)) {
        rate = (1.0 - amp_avg) * rate + amp_avg * ((double)nacc / (double)No);
    };
    // the records are private to this wavefront: a wavefront-level ordering
    // point is enough (SAIL_SWEEP_SYNC=1 selects a workgroup barrier; split sweeps,
    // whose records pass between wavefronts, have one there always)
    auto order = [&]() __attribute__((always_inline)) {
        if (wg_sync) __syncthreads();
        else wave_lds_sync();
    };

    if constexpr (SPLIT && WALK) {
        // Sec. 2.3 index selection (see below), split: what a walk draws does
        // not depend on the walker, so the stagers draw a batch of 16 proposals
        // with all their steps ahead.  The chain's lanes take one of a pair's
        // walks each, p's the even ones, s's the odd: the candidates' values are
        // read together, the steps decided one after another, and the pair's
        // table values read at its end.  A sweep's first batch is staged before
        // its move width is known: the chain completes those records.
        auto barrier = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        double *width = myrec + 2 * G * (kWalkRec + 2 * walk_len);
        auto wrec = [&](const int h, const int qq) __attribute__((always_inline)) { return myrec + (h * G + qq) * kWalkRec; };
        auto steps = [&](const int h, const int qq) __attribute__((always_inline)) {
            return (uint2 *)(myrec + 2 * G * kWalkRec) + (h * G + qq) * 2 * walk_len;
        };
        auto complete = [&](double *rc, const double ur) __attribute__((always_inline)) {
            const double rm1 = (1.0 - yeps * fma(2.0, ur, -1.0)) - 1.0;
            rc[0] = rm1;
            rc[1] = recip(rm1 + 1.0);
        };
        if (stager) {
            auto stage_walk = [&](const int h, const int q, const bool first) __attribute__((always_inline)) {
                uint32_t x2, x3, y0, y1, y2, y3;
                draw(q + c, k, op, os, x2, x3);
                double *rc = wrec(h, c);
                rc[0] = u01(x2);
                if (!first) complete(rc, u01(x2));
                rc[2] = staged_threshold(Tabs, u01(x3));
                rc[3] = __hiloint2double(os, op);
                uint2 *w = steps(h, c);
                for (int st = 0; st < walk_len; ++st) {
                    philox10((uint32_t)(q + c), (uint32_t)k, (uint32_t)lw, (uint32_t)(st + 1), key0, key1, y0, y1, y2, y3);
                    w[2 * st] = make_uint2((uint32_t)index_of(y0, No), y1);
                    w[2 * st + 1] = make_uint2((uint32_t)index_of(y2, No), y3);
                }
            };
            int h = 0;
            for (; k < k1; ++k) {
                temperature();
                for (q0 = 0; q0 < No; q0 += G) {
                    if (q0 > 0) yeps = *width;
                    stage_walk(h, q0, q0 == 0);
                    h ^= 1;
                    barrier();
                }
            }
            barrier();
            return;
        }
        __builtin_amdgcn_s_setprio(2);
        auto enter = [&]() __attribute__((always_inline)) {
            begin_sweep();
            if (c == 0) *width = yeps;
        };
        constexpr int W = 4;  // steps whose candidates are read together
        const int side = c & 1;
        auto step_words = [&](const int h, const int qq, const int st0, uint2 (&w)[W]) __attribute__((always_inline)) {
            const uint2 *p = steps(h, qq) + side;
#pragma unroll
            for (int t = 0; t < W; ++t) w[t] = p[2 * min(st0 + t, walk_len - 1)];
        };
        int h = 0;
        enter();
        barrier();
        for (;;) {
            if (q0 == 0) {
                double *rc = wrec(h, c);
                complete(rc, rc[0]);
                wave_lds_sync();
            }
            const int nq = min(G, No - q0);
            uint2 w[W];
            double rcv[kWalkRec];
            step_words(h, 0, 0, w);
#pragma unroll
            for (int t = 0; t < kWalkRec; ++t) rcv[t] = wrec(h, 0)[t];
            for (int qq = 0; qq < nq; ++qq) {
                Rec v;
                v.rm1 = rcv[0];
                v.rinv = rcv[1];
                v.thr = rcv[2];
                int x = side ? __double2hiint(rcv[3]) : __double2loint(rcv[3]);
                double gx = g * bsp[x];
                for (int st0 = 0;;) {
                    double cand[W];
#pragma unroll
                    for (int t = 0; t < W; ++t) cand[t] = bsp[w[t].x];
#pragma unroll
                    for (int t = 0; t < W; ++t) {
                        const double gc = g * cand[t];
                        const bool take = (u01(w[t].y) * gx < gc) & (st0 + t < walk_len);
                        gx = take ? gc : gx;
                        x = take ? (int)w[t].x : x;
                    }
                    st0 += W;
                    if (st0 >= walk_len) break;
                    step_words(h, qq, st0, w);
                }
                const int p = dpp_swap<0xA0>(x), s = dpp_swap<0xF5>(x);  // quad_perm 0, 0, 2, 2 and 1, 1, 3, 3
                rows(p, s, v);
                Pair pr;
                load_pair(p, s, pr);
                const double bp = bsp[p], bs = bsp[s];
                // the next proposal's words arrive meanwhile
                const int qn = min(qq + 1, nq - 1);
                step_words(h, qn, 0, w);
#pragma unroll
                for (int t = 0; t < kWalkRec; ++t) rcv[t] = wrec(h, qn)[t];
                pair_terms(p, s, pr, v.rm1 + 1.0, v.dp, v.ds, v.s1, v.t);
                body(qq, v, bp, bs, 0);
                wave_lds_sync();
            }
            h ^= 1;
            q0 += G;
            bool last = false;
            if (q0 >= No) {
                end_sweep();
                last = k + 1 >= k1;
                if (!last) {
                    ++k;
                    q0 = 0;
                    enter();
                }
            }
            barrier();
            if (last) break;
        }
    } else if constexpr (SPLIT) {
        // Both roles pass the same barriers: one to start, and in every sweep
        // two for the first two batches' records and one per batch.  Records
        // are staged two batches ahead of the chain (a ring of three) within a
        // sweep, since their move width follows from the sweep before; bins are
        // drawn one batch further ahead, across sweeps (a ring of four).
        auto barrier = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        double *width = myrec + 3 * G * kRecWords + 4 * G;  // move width of the sweep
        // masks of the proposals' shared bins, [slot][proposal], one set per pair of wavefronts
        uint64_t *hits = (uint64_t *)(lds + wpb * RSTR) + ws / (64 / G) * split_hits(G);
        auto uniform = [](const uint64_t x) __attribute__((always_inline)) {
            return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32;
        };
        auto of_owner_word = [](const uint32_t x, const int t) __attribute__((always_inline)) {
            return (uint32_t)lane_of<G>((int)x, t);
        };
        int rs = 0, bsl = 0;                                 // slots of the next record and bins
        if (stager) {
            Pair pr, npr;
            draw(c, k, np_, ns_, nx2, nx3);
            load_pair(np_, ns_, npr);
            stage_bins(0, c, np_, ns_);
            bsl = 1;
            barrier();
            for (; k < k1; ++k) {
                temperature();
                yeps = *width;
                for (q0 = 0; q0 < No; q0 += G) {
                    op = np_;
                    os = ns_;
                    const uint32_t x2 = nx2, x3 = nx3;
                    pr = npr;
                    const bool ends = q0 + G >= No;
                    const int q1 = ends ? 0 : q0 + G;
                    draw(q1 + c, ends ? k + 1 : k, np_, ns_, nx2, nx3);
                    load_pair(np_, ns_, npr);
                    stage_bins(bsl, q1 + c, np_, ns_);
                    bsl = (bsl + 1) & 3;
                    if constexpr (!ALLB) {
                        // the walkers' lanes of this wavefront mirror the chain's
                        ops = (uint32_t)op | (uint32_t)os << 16;
                        nps = (uint32_t)np_ | (uint32_t)ns_ << 16;
#pragma unroll
                        for (int t = 0; t < G; ++t) {
                            const uint32_t w = of_owner_word(ops, t);
                            const uint64_t h = shared_bins(t, (w & 0xffffu) * 0x10001u, (w >> 16) * 0x10001u);
                            if (lane == 0) hits[rs * G + t] = h;
                        }
                    }
                    stage(rs, q0 + c, op, os, x2, x3, pr);
                    rs = rs == 2 ? 0 : rs + 1;
                    barrier();
                }
                barrier();
                barrier();
            }
            return;
        }
        __builtin_amdgcn_s_setprio(2);
        // A bin's places: a resident one is read and stored in LDS, and its
        // memory offset is past the buffer, which costs no memory access;
        // another one's LDS slot is the one nothing reads.
        struct Place {
            uint32_t mem;
            double *lds;
        };
        auto place_of = [&](const int j) __attribute__((always_inline)) {
            if constexpr (!LDSB) return Place{brow + ((uint32_t)j << 3), nullptr};
            else return Place{j < nres ? kDropStore : brow + ((uint32_t)j << 3), bsp + min(j, nres)};
        };
        auto put = [&](const Place &o, const double x) __attribute__((always_inline)) {
            buffer_store_f64(b_rs, o.mem, x);
            if constexpr (LDSB) *o.lds = x;
        };
        Place opl, osl, npl, nsl;  // of op, os, np_ and ns_
        double lbp = 0.0, lbs = 0.0;
        auto load_next = [&](const double own_bins) __attribute__((always_inline)) {
            if constexpr (ALLB) return;
            np_ = __double2loint(own_bins);
            ns_ = __double2hiint(own_bins);
            npl = place_of(np_);
            nsl = place_of(ns_);
            nbp = buffer_load_f64(b_rs, npl.mem);
            nbs = buffer_load_f64(b_rs, nsl.mem);
            if constexpr (LDSB) {
                lbp = *npl.lds;
                lbs = *nsl.lds;
            }
        };
        begin_sweep();
        if (c == 0) *width = yeps;
        barrier();
        // Columns are loaded AHEAD proposals before they are used, their bins read
        // one proposal before that.  From memory they take longer than a proposal (32
        // jobs of 1300 bins, 300 walkers, FP64: 932 ns a proposal one ahead, 780 ns three;
        // alone, 5000 walkers, 389 and 345 ns; FP32, 2556 bins, 5000 walkers 350 and 285
        // ns).  As far as registers go: 8 FP64 values a lane two ahead, 16 lanes of FP64
        // or of more than 64 dimensions one.
        constexpr int AHEAD = LDSC ? 1 : G == 4 ? (M > 6 ? 2 : 3) : sizeof(R) == 4 && M <= 16 ? 3 : 1, V = AHEAD == 1 ? 2 : 4;
        static_assert(G % V == 0, "a batch turns the ring");
        Rec v[V];
        double next_bins;
        {
            // the first batch's bins and spectrum values
            const double own_bins = *bins_at(0, c);
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) {
                const double w0 = *bins_at(0, t);
                rows(__double2loint(w0), __double2hiint(w0), v[t]);
            }
            next_bins = *bins_at(0, AHEAD);
            load_next(own_bins);
        }
        for (;;) {
            barrier();
            barrier();
            fetch(rec_at(rs, 0), v[0]);
            bool last = false;
            for (q0 = 0; q0 < No; q0 += G) {
                const int bn = (bsl + 1) & 3, rn = rs == 2 ? 0 : rs + 1;  // the next batch's slots
                const bool ends = q0 + G >= No;
                // the batch's masks, read at its start, or at use (FP32, 16 lanes:
                // 221 against 231 ns a proposal; FP64: 220 against 215)
                constexpr bool HIT_AHEAD = G == 4 || sizeof(R) == 8;
                uint64_t hit[G] = {};
                if constexpr (!ALLB) {
                    const double own_bins = *bins_at(bn, c);
                    if constexpr (HIT_AHEAD) {
#pragma unroll
                        for (int t = 0; t < G; ++t) hit[t] = uniform(hits[rs * G + t]);
                    }
                    // this batch's spectrum values have arrived (waited for before
                    // the stores below are issued, so that nothing waits for those)
                    asm volatile("" : "+v"(nbp), "+v"(nbs));
                    if (__builtin_amdgcn_inverse_ballot_w64(accm & validm)) {
                        put(opl, obp);
                        put(osl, obs);
                    }
                    if constexpr (LDSB) {
                        nbp = npl.mem == kDropStore ? lbp : nbp;
                        nbs = nsl.mem == kDropStore ? lbs : nbs;
                    }
                    obp = fp ? fbp : nbp;
                    obs = fs ? fbs : nbs;
                    fp = fs = 0;
                    asm volatile("" : "+v"(fp), "+v"(fs));
                    accm = 0;
                    op = np_;
                    os = ns_;
                    opl = npl;
                    osl = nsl;
                    load_next(own_bins);
                    ops = (uint32_t)op | (uint32_t)os << 16;
                    nps = (uint32_t)np_ | (uint32_t)ns_ << 16;
                }
#pragma unroll
                for (int t = 0; t < G; ++t) {
                    // columns of a proposal to come (its bins were read a proposal
                    // ago), the next one's record, and the bins of the one whose
                    // columns are next
                    Rec &cur = v[t % V], &nx = v[(t + 1) % V], &far = v[(t + AHEAD) % V];
                    // (FP32: the spectrum values before the next proposal's words,
                    // which the decision would else wait behind, 200 to 192 ns a
                    // proposal; FP64 is as fast either way)
                    constexpr bool EARLY = ALLB && sizeof(R) == 4;
                    const double bp = EARLY ? bsp[cur.p] : 0.0, bs = EARLY ? bsp[cur.s] : 0.0;
                    rows(__double2loint(next_bins), __double2hiint(next_bins), far);
                    fetch(t + 1 < G ? rec_at(rs, t + 1) : rec_at(rn, 0), nx);
                    constexpr int B = AHEAD + 1;
                    next_bins = t + B < G ? *bins_at(bsl, t + B) : *bins_at(bn, t + B - G);
                    if constexpr (ALLB) {
                        if constexpr (EARLY) body(t, cur, bp, bs, 0);
                        else body(t, cur, bsp[cur.p], bsp[cur.s], 0);
                        wave_lds_sync();
                    } else {
                        if constexpr (!HIT_AHEAD) hit[t] = uniform(hits[rs * G + t]);
                        body(t, cur, obp, obs, hit[t]);
                    }
                    // keep each proposal's code together (bounds register pressure)
                    __builtin_amdgcn_sched_barrier(0);
                }
                rs = rn;
                bsl = bn;
                if (ends) {
                    end_sweep();
                    last = k + 1 >= k1;
                    if (!last) {
                        ++k;
                        begin_sweep();
                        if (c == 0) *width = yeps;
                    }
                }
                barrier();
            }
            if (last) break;
        }
        if constexpr (!ALLB) {
            if (__builtin_amdgcn_inverse_ballot_w64(accm & validm)) {
                put(opl, obp);
                put(osl, obs);
            }
        }
    } else if constexpr (WALK) {
        // Sec. 2.3 index selection: from the uniform p, s of each proposal,
        // walk_len independence Metropolis steps on a_j / A with uniform
        // proposals (step st draws Philox block (q, k, l, st): word 0 proposes
        // p, word 1 accepts it, words 2 and 3 the same for s), then the move of
        // the chosen pair.  The steps' draws and spectrum values do not depend
        // on one another: lane c takes step c + 1 (+ G, ...), and the lanes
        // exchange them through LDS.
        double *wk = myrec + G * (kRecWords + 1);
        for (; k < k1; ++k) {
            begin_sweep();
            for (q0 = 0; q0 < No; q0 += G) {
                Pair pr;
                uint32_t x2, x3;
                draw(q0 + c, k, op, os, x2, x3);
                stage_bins(0, q0 + c, op, os);
                stage(0, q0 + c, op, os, x2, x3, pr);
                order();
                const int nq = min(G, No - q0);
                for (int qq = 0; qq < nq; ++qq) {
                    Rec v;
                    fetch(rec_at(0, qq), v);
                    const double w0 = *bins_at(0, qq);
                    int p = __double2loint(w0), s = __double2hiint(w0);
                    double bp = load_b(p), bs = load_b(s);
                    for (int st0 = 0; st0 < walk_len; st0 += G) {
                        const int n = min(G, walk_len - st0);
                        if (c < n) {
                            uint32_t y0, y1, y2, y3;
                            philox10((uint32_t)(q0 + qq), (uint32_t)k, (uint32_t)lw, (uint32_t)(st0 + c + 1), key0, key1,
                                     y0, y1, y2, y3);
                            const int pc = index_of(y0, No), sc = index_of(y2, No);
                            double *w = wk + c * kWalkWords;
                            w[0] = __hiloint2double(sc, pc);
                            w[1] = load_b(pc);
                            w[2] = load_b(sc);
                            w[3] = u01(y1);
                            w[4] = u01(y3);
                        }
                        order();
                        for (int st = 0; st < n; ++st) {
                            const double *w = wk + st * kWalkWords;
                            const double bpc = w[1], bsc = w[2];
                            if (w[3] * (g * bp) < g * bpc) {
                                p = __double2loint(w[0]);
                                bp = bpc;
                            }
                            if (w[4] * (g * bs) < g * bsc) {
                                s = __double2hiint(w[0]);
                                bs = bsc;
                            }
                        }
                        order();
                    }
                    rows(p, s, v);
                    load_pair(p, s, pr);
                    pair_terms(p, s, pr, v.rm1 + 1.0, v.dp, v.ds, v.s1, v.t);
                    body(qq, v, bp, bs, 0);
                    order();
                }
            }
            end_sweep();
        }
    } else {
        // Three batches are under way: n runs, n + 1 has its bins, its spectrum
        // values load (where spectra are in memory) and its records are staged,
        // n + 2 is drawn and its table values load.  The work on the later two
        // stands between the loads and the serial tails of batch n's proposals
        // and fills their latencies.  After the last batch the draws are not
        // used.
        Pair npr, mpr;
        int mp = 0, ms_ = 0;
        uint32_t mx2 = 0, mx3 = 0;
        begin_sweep();
        draw(c, k, np_, ns_, nx2, nx3);
        if constexpr (!LDSB) {
            nbp = load_b(np_);
            nbs = load_b(ns_);
        }
        load_pair(np_, ns_, npr);
        int q1 = G < No ? G : 0, kn = G < No ? k : k + 1;  // the batch after the current one
        draw(q1 + c, kn, mp, ms_, mx2, mx3);
        load_pair(mp, ms_, mpr);
        stage_bins(0, c, np_, ns_);
        stage(0, c, np_, ns_, nx2, nx3, npr);
        order();
        Rec v[2];
        double next_bins;  // of the proposal after the next
        {
            const double w0 = *bins_at(0, 0);
            next_bins = *bins_at(0, 1);
            rows(__double2loint(w0), __double2hiint(w0), v[0]);
            fetch(rec_at(0, 0), v[0]);
        }
        for (;;) {
            if constexpr (!LDSB) {
                // this batch's spectrum values have arrived (waited for before
                // the stores below are issued, so that nothing waits for those)
                asm volatile("" : "+v"(nbp), "+v"(nbs));
                if (__builtin_amdgcn_inverse_ballot_w64(accm & validm)) {
                    buffer_store_f64(b_rs, brow + ((uint32_t)op << 3), obp);
                    buffer_store_f64(b_rs, brow + ((uint32_t)os << 3), obs);
                }
                obp = fp ? fbp : nbp;
                obs = fs ? fbs : nbs;
                fp = fs = 0;
                asm volatile("" : "+v"(fp), "+v"(fs));
                accm = 0;
            }
            op = np_;
            os = ns_;
            np_ = mp;
            ns_ = ms_;
            nx2 = mx2;
            nx3 = mx3;
            npr = mpr;
            if constexpr (!LDSB) {
                ops = (uint32_t)op | (uint32_t)os << 16;
                nps = (uint32_t)np_ | (uint32_t)ns_ << 16;
                nbp = load_b(np_);
                nbs = load_b(ns_);
            }
            const bool ends = q0 + G >= No;
            const int q2 = q1 + G >= No ? 0 : q1 + G, k2 = q1 + G >= No ? kn + 1 : kn;
#pragma unroll
            for (int t = 0; t < G; ++t) {
                // the next proposal's columns (its bins were read a proposal
                // ago), its record, and the bins of the one after it
                Rec &cur = v[t & 1], &nx = v[(t + 1) & 1];
                rows(__double2loint(next_bins), __double2hiint(next_bins), nx);
                fetch(t + 1 < G ? rec_at(buf, t + 1) : rec_at(buf ^ 1, 0), nx);
                next_bins = t + 2 < G ? *bins_at(buf, t + 2) : *bins_at(buf ^ 1, t + 2 - G);
                if (t == 0) {
                    stage_bins(buf ^ 1, q1 + c, np_, ns_);
                    stage(buf ^ 1, q1 + c, np_, ns_, nx2, nx3, npr);
                }
                if (t == 1) {
                    draw(q2 + c, k2, mp, ms_, mx2, mx3);
                    load_pair(mp, ms_, mpr);
                }
                if constexpr (LDSB) body(t, cur, bsp[cur.p], bsp[cur.s], 0);
                else body(t, cur, obp, obs, 0);
                if (t == 1) order();
                else if constexpr (LDSB) wave_lds_sync();
                // keep each proposal's code together (bounds register pressure)
                __builtin_amdgcn_sched_barrier(0);
            }
            if (ends) {
                end_sweep();
                if (kn >= k1) break;
                // the next sweep's temperature and move width: stage again
                k = kn;
                begin_sweep();
                stage(buf ^ 1, q1 + c, np_, ns_, nx2, nx3, npr);
                order();
                fetch(rec_at(buf ^ 1, 0), v[0]);
            }
            buf ^= 1;
            q0 = q1;
            q1 = q2;
            kn = k2;
        }
        if constexpr (!LDSB) {
            if (__builtin_amdgcn_inverse_ballot_w64(accm & validm)) {
                buffer_store_f64(b_rs, brow + ((uint32_t)op << 3), obp);
                buffer_store_f64(b_rs, brow + ((uint32_t)os << 3), obs);
            }
        }
    }
    if (valid) {
        if (c < CH) {
#pragma unroll
            for (int t = 0; t < MR; ++t) phig[t] = phi[t];
        }
        if constexpr (LDSB) {
            wave_lds_sync();
            double *bl = a.b + (size_t)l * No;
            for (int j = c; j < nres; j += G) bl[j] = bsp[j];
        }
        if (c == 0) {
            a.gsc[l] = g;
            a.ginv[l] = ginv;
            a.chi2[l] = chi2;
            a.rate[l] = rate;
        }
    }
}

// Workgroups of 64 to kSweepThreads threads (split sweeps: 128 to twice as
// many), as the launch plan asks.
constexpr int kSweepThreads = 256;

template <typename R, int M, int G, bool LDSC, bool LDSB, int MODE>
__global__ __launch_bounds__(kSweepThreads) void k_sweep(SweepArgs a)
{
    extern __shared__ __align__(16) double lds[];
    sweep_block<R, M, G, LDSC, LDSB, MODE, false>(a, blockIdx.x, lds);
}

template <typename R, int M, bool LDSC, bool LDSB>
__global__ __launch_bounds__(2 * kSweepThreads) void k_sweep_split(SweepArgs a)
{
    extern __shared__ __align__(16) double lds[];
    sweep_block<R, M, 4, LDSC, LDSB, kSweepFast, true>(a, blockIdx.x, lds);
}

template <typename R, int M, bool LDSC, bool LDSB, int MODE>
__global__ __launch_bounds__(2 * kSweepThreads) void k_sweep_split16(SweepArgs a)
{
    extern __shared__ __align__(16) double lds[];
    sweep_block<R, M, 16, LDSC, LDSB, MODE, true>(a, blockIdx.x, lds);
}

// Many problems in one launch: problem q owns workgroups [first[q], first[q + 1]).
// Traces (4 lanes a walker) and walks (8, or 4 in a large batch), 16 in a wide
// basis, columns and spectra in memory.
template <typename R, int M, int MODE, int G>
__global__ __launch_bounds__(kSweepThreads, 2) void k_sweep_batched(const SweepArgs *__restrict__ jobs,
                                                                   const int *__restrict__ first, int n_jobs)
{
    extern __shared__ __align__(16) double lds[];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    const int q = owner_of(first, n_jobs, b);
    sweep_block<R, M, G, false, false, MODE, false>(jobs[q], b - first[q], lds);
}

template <typename R, int M>
__global__ __launch_bounds__(2 * kSweepThreads) void k_sweep_split_batched(const SweepArgs *__restrict__ jobs,
                                                                          const int *__restrict__ first, int n_jobs, int near)
{
    extern __shared__ __align__(16) double lds[];
    const int b = near ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int q = owner_of(first, n_jobs, b);
    const SweepArgs &a = jobs[q];
    const int block = b - first[q];
    if constexpr (wide_basis(M)) {
        if (a.columns_lds) sweep_block<R, M, 16, true, false, kSweepFast, true>(a, block, lds);
        else sweep_block<R, M, 16, false, false, kSweepFast, true>(a, block, lds);
    }
    else if (a.lanes == 16) sweep_block<R, M, 16, true, false, kSweepFast, true>(a, block, lds);
    else if (a.resident) sweep_block<R, M, 4, true, true, kSweepFast, true>(a, block, lds);
    else if (a.columns_lds) sweep_block<R, M, 4, true, false, kSweepFast, true>(a, block, lds);
    else sweep_block<R, M, 4, false, false, kSweepFast, true>(a, block, lds);
}

// --------------------------------------------------------------------------
// Block reductions
// --------------------------------------------------------------------------
template <typename T, typename Op>
__device__ T block_reduce(T v, T *scratch, Op op)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = (blockDim.x + 63) >> 6;
    for (int m = 32; m >= 1; m >>= 1) v = op(v, __shfl_xor(v, m, 64));
    __syncthreads();
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    T r = scratch[0];
    for (int w = 1; w < nwaves; ++w) r = op(r, scratch[w]);
    __syncthreads();
    return r;
}

struct OpSum {
    template <typename T>
    __device__ T operator()(T x, T y) const { return x + y; }
};
struct OpMin {
    __device__ double operator()(double x, double y) const { return fmin(x, y); }
};
struct OpMax {
    __device__ double operator()(double x, double y) const { return fmax(x, y); }
};

__device__ __forceinline__ int lane_read(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ double lane_read(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Reduction over the 64 lanes of a full wavefront without LDS: DPP steps
// within each 16-lane row, then the four row results read as scalars.
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op)
{
    v = op(v, dpp_swap<0xB1>(v));   // lane ^ 1
    v = op(v, dpp_swap<0x4E>(v));   // lane ^ 2
    v = op(v, dpp_swap<0x141>(v));  // row_half_mirror
    v = op(v, dpp_swap<0x140>(v));  // row_mirror
    return op(op(lane_read(v, 0), lane_read(v, 16)), op(lane_read(v, 32), lane_read(v, 48)));
}

// --------------------------------------------------------------------------
// Resync: imprint or smooth, fold the lazy scale, optionally renormalise both
// sums, recompute the walkers' coordinates and chi^2 (8 or 16 walkers a workgroup).
// --------------------------------------------------------------------------
struct ResyncArgs {
    int n_omega, n_tau;
    int cols;             // columns of E: n_tau, then 4 echunk
    int echunk, chunk;    // basis dimensions per chunk as stored in E and in phi
    const double *omega;
    const double *E;      // [N_omega][cols] e^{-omega_j tau_i}, then the column in the basis
    const double *wh, *Phit;
    double *b, *gsc, *ginv, *chi2;
    void *phi;                   // [N_w][4][chunk], in the loop precision
    double A, B;
    int renorm;
    const int32_t *list;        // optional walker list
    const int32_t *list_count;  // its length (device)
    int n_items;                // walkers to resync when there is no list
    const int32_t *donors;      // optional, parallel to list: imprint a <- t a_donor + (1 - t) a first
    double imprint_t;
    const double *imprint_t_dev;  // optional: the imprint strength in device memory (adaptive branching)
    double smooth;              // > 0: three-point smoothing (Sec. 2.6) before the renormalisation
    unsigned int *watch;        // optional watchdog flag: bit 0 drift above watch_bound, bit 1 non-finite chi^2
    double watch_bound;         // relative sum-rule drift allowed before the renormalisation
    double *drift;              // optional [N_w]: each walker's relative sum-rule drift before the renormalisation
};

// Doubles between two walkers' spectra in the resync's LDS: odd, so that the 16
// rows a matrix instruction reads lie in different banks (but for the largest
// N_omega that fits, which needs every word).
constexpr int kResyncMost = 2556;
__host__ __device__ constexpr int resync_stride(int n_omega) { return n_omega < kResyncMost ? n_omega | 1 : n_omega; }


__device__ __forceinline__ double wave_sum(double v)
{
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// Calls use(r, i, v) with v the product of walker slot lane / 16 + 4 r's spectrum
// (sb, WPB rows of `ld` in LDS) and column i < n of E (rows of `cols`), in FP64 on
// the matrix cores: a wavefront takes up to three tiles of 16 columns at a time.
// 8 walkers leave half of a tile's rows idle.
template <int WPB, typename F>
__device__ __forceinline__ void columns_product(const double *sb, const int ld, const int No, const double *E, const int cols,
                                                const int n, F &&use)
{
    // lane: column lane % 16 of a tile; rows (walkers) and bins by lane / 16
    constexpr int T = 3;  // tiles at a time
    typedef double v4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lc = lane & 15, lk = lane >> 4;
    const double *arow = sb + (lc % WPB) * ld;
    const int tiles = (n + 15) / 16;
    for (int t0 = wave; t0 < tiles; t0 += 4 * T) {
        v4 acc[T] = {};
        int col[T];
#pragma unroll
        for (int t = 0; t < T; ++t) col[t] = min((t0 + 4 * t) * 16 + lc, n - 1);  // past the last: not used
        int k = lk;
        for (; k - lk + 16 <= No; k += 16) {
            double av[4], e[4][T];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                av[u] = arow[k + 4 * u];
                const double *Er = E + (size_t)(k + 4 * u) * cols;
#pragma unroll
                for (int t = 0; t < T; ++t) e[u][t] = Er[col[t]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], e[u][t], acc[t], 0, 0, 0);
        }
        for (; k - lk < No; k += 4) {
            const bool in = k < No;
            const double av = in ? arow[k] : 0.0;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double e = in ? E[(size_t)k * cols + col[t]] : 0.0;
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, e, acc[t], 0, 0, 0);
            }
        }
        // acc[t][r]: walker slot lk + 4 r, column i
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int i = (t0 + 4 * t) * 16 + lc;
            if (i >= n) continue;
#pragma unroll
            for (int r = 0; r < WPB / 4; ++r) use(r, i, acc[t][r]);
        }
    }
}

// WPB (8 or 16) walkers per workgroup.  The columns, and the basis coordinates
// beside them, are a product [walkers x N_omega] [N_omega x cols] in FP64 on the
// matrix cores: a wavefront takes up to three tiles of 16 columns at a time, the
// walkers' spectra come from LDS and E from the caches.  Phi_i's residuals give
// chi^2; the basis coordinates are stored in the loop precision R.  A walker's
// sums are taken in the same order for either WPB.  8 walkers leave half of a
// tile's rows idle but twice the workgroups.  512 bins, 144 columns, 16384 walkers:
// 93 us, 26 TFLOP/s (165 us on the vector units, which an LDS read per FMA held
// back); 64 walkers of 64 bins 11 us (19), mostly latency.
template <typename R, int WPB>
__device__ __forceinline__ void resync_block(const ResyncArgs &a, const int block, double *sh)
{
    // sh: [WPB][stride] spectra, then [4][WPB] partial residues
    const int No = a.n_omega, Nt = a.n_tau, cols = a.cols, ld = resync_stride(No);
    double *sb = sh;
    double *red = sh + (size_t)WPB * ld;
    const int count = a.list ? *a.list_count : a.n_items;
    const int base = block * WPB;
    if (base >= count) return;
    int wl[WPB];
#pragma unroll
    for (int w = 0; w < WPB; ++w) {
        const int idx = base + w;
        wl[w] = idx < count ? (a.list ? a.list[idx] : idx) : -1;
    }
    // imprint (Sec. 2.5; donors are never targets, so their spectra are
    // read-only here), then fold the lazy scale
#pragma unroll
    for (int w = 0; w < WPB; ++w) {
        if (wl[w] < 0) continue;
        const double g = a.gsc[wl[w]];
        const double *bl = a.b + (size_t)wl[w] * No;
        if (a.donors) {
            const double t = a.imprint_t_dev ? *a.imprint_t_dev : a.imprint_t, t1 = 1.0 - t;
            const double *bd = a.b + (size_t)a.donors[base + w] * No;
            for (int j = threadIdx.x; j < No; j += blockDim.x) sb[w * ld + j] = g * (t * bd[j] + t1 * bl[j]);
        } else {
            for (int j = threadIdx.x; j < No; j += blockDim.x) sb[w * ld + j] = g * bl[j];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (a.smooth > 0.0) {
        // Sec. 2.6 stencil on the values before the update: each wavefront
        // sweeps its walkers' rows in chunks of 64 lanes, carrying the old
        // value left of the chunk in a register (the wavefront's LDS reads of
        // a chunk precede its writes, and the next chunk's reads lie beyond)
        const double sm = a.smooth, cm = 1.0 - 2.0 * sm, em = 1.0 - sm;
        for (int w = wave; w < WPB; w += kThreads / 64) {
            if (wl[w] < 0) continue;
            double *row = sb + w * ld;
            double left = 0.0;
            for (int j0 = 0; j0 < No; j0 += 64) {
                const int j = j0 + lane;
                const double cur = j < No ? row[j] : 0.0;
                const double right = j + 1 < No ? row[j + 1] : 0.0;
                double prev = __shfl_up(cur, 1, 64);
                if (lane == 0) prev = left;
                left = __shfl(cur, 63, 64);
                double v;
                if (j == 0) v = em * cur + sm * right;
                else if (j == No - 1) v = em * cur + sm * prev;
                else v = sm * prev + cm * cur + sm * right;
                wave_lds_sync();
                if (j < No) row[j] = v;
            }
        }
        __syncthreads();
    }
    if (a.renorm) {
        // Reading of Sec. 2.6: a_j <- a_j (1 + d0 + d1 omega_j) restores both sums
        // 16 lanes a walker, every walker at once
        const int w = threadIdx.x >> 4, c = threadIdx.x & 15;
        int walker = -1;
#pragma unroll
        for (int t = 0; t < WPB; ++t) walker = w == t ? wl[t] : walker;
        if (walker >= 0) {
            double *row = sb + w * ld;
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
            for (int j = c; j < No; j += 16) {
                const double v = row[j], x = a.omega[j];
                s0 += v;
                s1 += v * x;
                s2 += v * x * x;
            }
            s0 = group_sum<16>(s0);
            s1 = group_sum<16>(s1);
            s2 = group_sum<16>(s2);
            if ((a.watch || a.drift) && c == 0) {
                // both sums are invariants of every move (Sec. 2.2): their drift
                // since the last renormalisation measures accumulated error
                const double drift = fmax(fabs(s0 - a.A) / a.A, fabs(s1 - a.B) / fabs(a.B));
                if (a.watch && !(drift <= a.watch_bound)) atomicOr(a.watch, 1u);
                if (a.drift) a.drift[walker] = drift;
            }
            const double e0 = a.A - s0, e1 = a.B - s1;
            const double det = s0 * s2 - s1 * s1;
            if (det > 0.0 && isfinite(det)) {
                const double d0 = (e0 * s2 - e1 * s1) / det;
                const double d1 = (e1 * s0 - e0 * s1) / det;
                for (int j = c; j < No; j += 16) row[j] = row[j] + row[j] * (d0 + d1 * a.omega[j]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int w = 0; w < WPB; ++w) {
        if (wl[w] < 0) continue;
        double *bl = a.b + (size_t)wl[w] * No;
        for (int j = threadIdx.x; j < No; j += blockDim.x) bl[j] = sb[w * ld + j];
        if (threadIdx.x == 0) {
            a.gsc[wl[w]] = 1.0;
            a.ginv[wl[w]] = 1.0;
        }
    }
    double part[WPB / 4] = {};
    int mine[WPB / 4];  // the walkers of this lane's results
    const int lc = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int r = 0; r < WPB / 4; ++r) {
        mine[r] = -1;
#pragma unroll
        for (int w = 0; w < WPB; ++w) mine[r] = lk + 4 * r == w ? wl[w] : mine[r];
    }
    columns_product<WPB>(sb, ld, No, a.E, cols, cols, [&](const int r, const int i, const double v) __attribute__((always_inline)) {
        const int walker = mine[r];
        if (walker < 0) return;
        if (i < Nt) {
            const double rsd = v - a.Phit[i];
            part[r] += a.wh[i] * rsd * rsd;
        } else {
            const int d = i - Nt, q = d / a.echunk, x = d % a.echunk;
            if (x < a.chunk) ((R *)a.phi)[((size_t)walker * 4 + q) * a.chunk + x] = (R)v;
        }
    });
#pragma unroll
    for (int r = 0; r < WPB / 4; ++r) {
        const double v = group_sum<16>(part[r]);
        if (lc == 0) red[wave * WPB + lk + 4 * r] = v;
    }
    __syncthreads();
    if (threadIdx.x < WPB) {
        int walker = -1;
#pragma unroll
        for (int w = 0; w < WPB; ++w) walker = (int)threadIdx.x == w ? wl[w] : walker;
        if (walker >= 0) {
            double v = 0.0;
            for (int wv = 0; wv < kThreads / 64; ++wv) v += red[wv * WPB + threadIdx.x];
            a.chi2[walker] = v;
            if (a.watch && !isfinite(v)) atomicOr(a.watch, 2u);
        }
    }
}

template <typename R, int WPB>
__global__ __launch_bounds__(kThreads) void k_resync(ResyncArgs a)
{
    extern __shared__ double sh[];
    resync_block<R, WPB>(a, blockIdx.x, sh);
}

template <typename R, int WPB>
__global__ __launch_bounds__(kThreads) void k_resync_batched(const ResyncArgs *__restrict__ jobs,
                                                             const int *__restrict__ first, int n_jobs)
{
    extern __shared__ double sh[];
    const int q = owner_of(first, n_jobs, blockIdx.x);
    resync_block<R, WPB>(jobs[q], blockIdx.x - first[q], sh);
}

// Reconstructions of `n` walkers for read-out: F_i = c_i Phi_i, Phi_i = sum_j a_j E_ji
// rounded to the loop precision, as the resync's product (512 bins, 128 times, 16384
// walkers: 126 us in two launches; the read-out of the whole state 9.2 ms, 14.1 ms with a
// workgroup per walker, a serial sum per time and the host's loops over the rows).
template <typename R, int WPB>
__global__ __launch_bounds__(kThreads) void k_reconstruct(int n, int n_omega, int n_tau, int cols, const double *E,
                                                          const double *cfac, const double *b, const double *gsc, double *F)
{
    extern __shared__ double sh[];
    const int ld = resync_stride(n_omega), base = blockIdx.x * WPB;
    for (int w = 0; w < WPB && base + w < n; ++w) {
        const double g = gsc[base + w];
        const double *bl = b + (size_t)(base + w) * n_omega;
        for (int j = threadIdx.x; j < n_omega; j += kThreads) sh[w * ld + j] = g * bl[j];
    }
    __syncthreads();
    const int lk = (threadIdx.x & 63) >> 4;
    columns_product<WPB>(sh, ld, n_omega, E, cols, n_tau, [&](const int r, const int i, const double v) __attribute__((always_inline)) {
        const int l = base + lk + 4 * r;
        if (l < n) F[(size_t)l * n_tau + i] = cfac[i] * (double)(R)v;
    });
}

// --------------------------------------------------------------------------
// Tables of a problem, one workgroup per bin: the exact column E_j, its terms
// D_j = sum_i w_i K_ij^2 and V_j = sum_i c_i K_ij, and its coordinates along up
// to kBasisPass basis vectors (`proj`, times sqrt(wh)).  Latency and the FP64
// exponentials bound it: creating a problem of 512 bins and 128 times takes 0.33 ms,
// of 1024 and 256 0.52 ms (1.34 and 4.3 ms with the exponentials on the host).
// --------------------------------------------------------------------------
constexpr int kBasisPass = 32;
struct TableArgs {
    int n_omega, n_tau;
    int d0, nd;           // first basis vector of the pass, and how many
    const double *omega, *tau, *wh, *cn;
    const double *proj;   // [nd][n_tau]
    double *tail;         // [n_omega] squared coordinates of a column from vector d0 on, relative to its norm
    double *worst;        // [nd] the largest tail from each of the vectors on
    double *E;            // written if not NULL: [n_omega][cols], and bin
    double4 *bin;
    int cols, echunk;
};

__global__ __launch_bounds__(kThreads) void k_tables(TableArgs a)
{
    extern __shared__ __align__(16) double lds[];
    __shared__ double part[2][kThreads / 64], cs[kBasisPass];
    const int j = blockIdx.x, Nt = a.n_tau;
    const double w = a.omega[j];
    double D = 0.0, V = 0.0;
    for (int i = threadIdx.x; i < Nt; i += kThreads) {
        const double e = exp(-w * a.tau[i]);
        lds[i] = e;
        D += a.wh[i] * e * e;
        V += a.cn[i] * e;
    }
    D = wave_sum(D);
    V = wave_sum(V);
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = D;
        part[1][threadIdx.x >> 6] = V;
    }
    __syncthreads();
    D = V = 0.0;
    for (int t = 0; t < kThreads / 64; ++t) {
        D += part[0][t];
        V += part[1][t];
    }
    const bool spans = D > 0.0 && isfinite(D);  // a column that overflows or vanishes spans nothing
    const int c = threadIdx.x & 15;
    for (int d = threadIdx.x >> 4; d < a.nd; d += kThreads / 16) {
        const double *q = a.proj + (size_t)d * Nt;
        double v = 0.0;
        for (int i = c; i < Nt; i += 16) v = fma(lds[i], q[i], v);
        v = group_sum<16>(v);
        if (c == 0) cs[d] = spans ? v : 0.0;
    }
    __syncthreads();
    if (a.E) {
        double *row = a.E + (size_t)j * a.cols;
        if (a.d0 == 0) {
            for (int i = threadIdx.x; i < a.cols; i += kThreads) row[i] = i < Nt ? lds[i] : 0.0;
            if (threadIdx.x == 0) a.bin[j] = make_double4(w, D, V, 0.0);
        }
        __syncthreads();
        for (int d = threadIdx.x; d < a.nd; d += kThreads)
            row[Nt + ((a.d0 + d) & 3) * a.echunk + ((a.d0 + d) >> 2)] = cs[d];
    } else if ((int)threadIdx.x < a.nd) {
        // (an earlier pass's maxima may stay: tails only grow towards the first
        // vector; a read first spares most of the atomics)
        const int d = threadIdx.x;
        double t = a.tail[j];
        for (int e = a.nd - 1; e >= d && spans; --e) t += cs[e] * cs[e] / D;
        if (spans && t > a.worst[d])
            atomicMax((unsigned long long *)&a.worst[d], (unsigned long long)__double_as_longlong(t));
        wave_lds_sync();  // (nd <= 64: one wavefront has read the tail)
        if (d == 0) a.tail[j] = spans ? t : 1.0;
    }
}

// (G_k, H_k) = sum_i w_i (1, tau_i) e^{-wbar_k tau_i}, a wavefront per pair sum.
__global__ __launch_bounds__(64) void k_pair_sums(int n_tau, double w0x2, double dW, const double *tau, const double *wh,
                                                  double2 *GH)
{
    const double wbar = w0x2 + (double)blockIdx.x * dW;
    double g = 0.0, h = 0.0;
    for (int i = threadIdx.x; i < n_tau; i += 64) {
        const double e = wh[i] * exp(-wbar * tau[i]);
        g += e;
        h += e * tau[i];
    }
    g = wave_sum(g);
    h = wave_sum(h);
    if (threadIdx.x == 0) GH[blockIdx.x] = make_double2(g, h);
}

// The basis columns of E in the loop precision, [N_omega][4][chunk].
template <typename R>
__global__ __launch_bounds__(kThreads) void k_columns(int n, int n_tau, int cols, int echunk, int chunk, const double *E, R *col)
{
    const int x = blockIdx.x * kThreads + threadIdx.x;
    if (x >= n) return;
    const int t = x % chunk, q = x / chunk & 3, j = x / (4 * chunk);
    col[x] = t < echunk ? (R)E[(size_t)j * cols + n_tau + q * echunk + t] : (R)0;
}

__global__ void k_init_walkers(int n_walkers, int n_omega, const double *a0, double *b, double *gsc, double *ginv,
                               double *rate)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)n_walkers * n_omega;
    if (idx < total) b[idx] = a0[idx % n_omega];
    if (idx < (size_t)n_walkers) {
        gsc[idx] = 1.0;
        ginv[idx] = 1.0;
        rate[idx] = 1.0;
    }
}

// Watchdog bookkeeping, w = {flag, snapshot sweep, trip sweep}: the walker
// state is copied to the snapshot only while no check has tripped.
__global__ void k_watch_reset(unsigned int *w, int k)
{
    w[0] = 0u;
    w[1] = (unsigned int)k;
    w[2] = 0xffffffffu;
}

// One record of the per-block log: population statistics after the block's
// resync (and branching event, if any), reduced by one workgroup in a fixed
// order, so the record is deterministic.
static_assert(sizeof(sail_block_record) == 64, "block record layout");
struct BlockLogArgs {
    int n;
    const double *chi2, *rate, *drift;  // drift may be null (no renormalising resync at this boundary)
    const double *Tabs;
    int sweep, event;
    sail_block_record *out;
};

// The rank-th smallest of n keys in LDS (residue bit patterns: residues are
// >= 0, so their bits order like their values; a NaN sorts last): a radix
// select in 8-bit digits from bit shift0 down, among the keys that match
// prefix on mask (the bits above shift0 + 8, common to all keys), one
// histogram in LDS per digit.
__device__ double block_select(const uint64_t *keys, int n, int rank, int shift0, uint64_t prefix, uint64_t mask,
                               unsigned int *hist, uint64_t *sh_prefix, int *sh_k)
{
    static_assert(kThreads == 256, "one histogram bin per thread");
    int k = rank;
    for (int shift = shift0; shift >= 0; shift -= 8) {
        hist[threadIdx.x] = 0u;
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += kThreads) {
            const uint64_t key = keys[i];
            if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        // inclusive prefix sum of the bins (one per thread, in place); the
        // digit is the bin whose range of ranks holds k, and the keys that
        // match the prefix number more than k, so exactly one bin holds it
        const unsigned int own = hist[threadIdx.x];
        unsigned int incl = own;
        for (int d = 1; d < kThreads; d <<= 1) {
            const unsigned int add = (int)threadIdx.x >= d ? hist[threadIdx.x - d] : 0u;
            __syncthreads();
            incl += add;
            hist[threadIdx.x] = incl;
            __syncthreads();
        }
        if (incl - own <= (unsigned int)k && (unsigned int)k < incl) {
            *sh_k = k - (int)(incl - own);
            *sh_prefix = prefix | ((uint64_t)threadIdx.x << shift);
        }
        __syncthreads();
        k = *sh_k;
        prefix = *sh_prefix;
        mask |= (uint64_t)255 << shift;
        __syncthreads();  // every thread has read the digit before the histogram is cleared
    }
    return __longlong_as_double((long long)prefix);
}

constexpr int kLogKeys = kBranchMaxWalkers;  // residues a record's LDS holds (every runnable population)

__device__ __forceinline__ void block_record(const BlockLogArgs &a)
{
    __shared__ uint64_t keys[kLogKeys];  // the residues' bit patterns (sign cleared)
    __shared__ unsigned int hist[kThreads];
    __shared__ uint64_t sel_prefix;
    __shared__ int sel_k;
    __shared__ double red[4][kThreads];
    __shared__ double dred[kThreads];
    __shared__ uint64_t kred[2][kThreads];
    const int n = a.n;
    double mn = INFINITY, mx = -INFINITY, sum = 0.0, rsum = 0.0, dmax = 0.0;
    uint64_t kmin = ~0ull, kmax = 0ull;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += kThreads) {
        const double c = a.chi2[i];
        mn = fmin(mn, c);
        mx = fmax(mx, c);
        sum += c;
        rsum += a.rate[i];
        if (a.drift) {
            const double d = a.drift[i];
            dmax = fmax(dmax, isnan(d) ? INFINITY : d);  // a drift that is not a number shows as infinite
        }
        const uint64_t key = (uint64_t)__double_as_longlong(c) & 0x7FFFFFFFFFFFFFFFull;
        if (i < kLogKeys) keys[i] = key;
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
    }
    red[0][threadIdx.x] = sum;
    red[1][threadIdx.x] = rsum;
    red[2][threadIdx.x] = mn;
    red[3][threadIdx.x] = mx;
    dred[threadIdx.x] = dmax;
    kred[0][threadIdx.x] = kmin;
    kred[1][threadIdx.x] = kmax;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            const int j = threadIdx.x + h;
            red[0][threadIdx.x] += red[0][j];
            red[1][threadIdx.x] += red[1][j];
            red[2][threadIdx.x] = fmin(red[2][threadIdx.x], red[2][j]);
            red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][j]);
            dred[threadIdx.x] = fmax(dred[threadIdx.x], dred[j]);
            kred[0][threadIdx.x] = kred[0][j] < kred[0][threadIdx.x] ? kred[0][j] : kred[0][threadIdx.x];
            kred[1][threadIdx.x] = kred[1][j] > kred[1][threadIdx.x] ? kred[1][j] : kred[1][threadIdx.x];
        }
        __syncthreads();
    }
    // median as numpy takes it: the middle residue, or the mean of the two.
    // Every key lies between the smallest and the largest, so the bits above
    // their highest differing digit are common to all and the select starts
    // below them.
    const uint64_t klo = kred[0][0], khi = kred[1][0];
    double median;
    if (n > kLogKeys) {
        median = NAN;  // not reached: runs take at most kLogKeys walkers
    } else if (klo == khi) {
        median = __longlong_as_double((long long)klo);
    } else {
        const int top = 63 - __clzll((long long)(klo ^ khi));
        const int shift0 = (top / 8) * 8;
        const uint64_t mask = shift0 + 8 >= 64 ? 0ull : ~((1ull << (shift0 + 8)) - 1ull);
        const uint64_t prefix = klo & mask;
        const double med_hi = block_select(keys, n, n / 2, shift0, prefix, mask, hist, &sel_prefix, &sel_k);
        if (n & 1) {
            median = med_hi;
        } else {
            // the residue of rank n/2 - 1: the upper middle itself when fewer
            // than n/2 residues lie below it, else the largest one below it
            const uint64_t khm = (uint64_t)__double_as_longlong(med_hi);
            uint64_t below = 0ull;
            unsigned int cnt = 0u;
            for (int i = threadIdx.x; i < n; i += kThreads) {
                const uint64_t key = keys[i];
                if (key < khm) {
                    ++cnt;
                    below = key > below ? key : below;
                }
            }
            kred[0][threadIdx.x] = below;
            hist[threadIdx.x] = cnt;
            __syncthreads();
            for (int h = kThreads / 2; h > 0; h >>= 1) {
                if ((int)threadIdx.x < h) {
                    const int j = threadIdx.x + h;
                    kred[0][threadIdx.x] = kred[0][j] > kred[0][threadIdx.x] ? kred[0][j] : kred[0][threadIdx.x];
                    hist[threadIdx.x] += hist[j];
                }
                __syncthreads();
            }
            const uint64_t klm = hist[0] < (unsigned int)(n / 2) ? khm : kred[0][0];
            median = (__longlong_as_double((long long)klm) + med_hi) / 2.0;
        }
    }
    if (threadIdx.x == 0) {
        sail_block_record r;
        r.sweep = a.sweep;
        r.event = a.event;
        r.T = a.Tabs[a.sweep - 1];
        r.chi2_min = red[2][0];
        r.chi2_mean = red[0][0] / n;
        r.chi2_median = median;
        r.chi2_max = red[3][0];
        r.rate_mean = red[1][0] / n;
        r.drift_max = a.drift ? dred[0] : -1.0;
        *a.out = r;
    }
}

__global__ __launch_bounds__(kThreads) void k_block_record(BlockLogArgs a) { block_record(a); }

// many problems: workgroup b writes the record of problem b
__global__ __launch_bounds__(kThreads) void k_block_record_batched(const BlockLogArgs *__restrict__ args)
{
    block_record(args[blockIdx.x]);
}

__global__ void k_watch_mark(unsigned int *w, int k)
{
    if (w[0] == 0u) w[1] = (unsigned int)k;
    else if (w[2] == 0xffffffffu) w[2] = (unsigned int)k;
}

// Copies n 8-byte words; with w given, only while its flag is clear.
__global__ void k_watch_copy(const unsigned int *w, double *dst, const double *src, size_t n)
{
    if (w && w[0] != 0u) return;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// --------------------------------------------------------------------------
// Imprinted branching (Sec. 2.5).
//   w_l = exp[-(chi^2_l - P_r) Delta],  m_l = floor(w_l + xi_l);
// m_l reaches k once P_r >= theta_{l,k} = chi^2_l + ln(k - xi_l) / Delta, so
// sum m = N_w for P_r between the N_w-th and (N_w+1)-th smallest threshold
// (taken at their midpoint).  Delta: the smallest value of a fixed doubling +
// bisection search whose zero count reaches round(fraction N_w).
// One workgroup; walker l = thread * WPT + q.
// --------------------------------------------------------------------------
struct BranchArgs {
    int n;
    const double *chi2;
    uint32_t key0, key1, event;
    double fraction;
    const double *rate;   // running acceptance rates (adaptive branching)
    int adaptive;         // scale fraction and imprint strength by the mean rate
    double imprint_t;
    double *t_eff;        // optional: receives the event's imprint strength
    int32_t *m, *targets, *donors, *npairs;
    double *ev_delta, *ev_pr;
    int32_t *ev_z, *ev_status, *ev_m;  // ev_m optional, [event][n]
    double *ev_gap, *ev_bracket;       // margins of the solve (see branch_block)
};

// With y = e^{(P - chi^2_min) Delta} and w_l = e^{-(chi^2_l - chi^2_min) Delta},
// m_l(P) = #{k >= 1 : theta_{l,k} <= P} = floor(xi_l + y w_l): for a fixed
// Delta the w_l are computed once, and every count is one FMA per walker.
// Counts are capped at n + 1 (enough to decide against n).
__device__ __forceinline__ int branch_m(double xi, double w, double y, int n)
{
    const double v = fma(y, w, xi);
    if (!(v < (double)(n + 1))) return n + 1;
    return (int)v;
}

// Shapes of a branching workgroup, by the number of walkers.  An evaluation is
// a chain of counts, each a handful of instructions per walker and a
// reduction over the workgroup, so a small population takes few wavefronts
// (their barrier is what a count waits for; one wavefront needs none) and few
// walkers per thread (64 walkers, one event in one workgroup: 1250 us with 1024
// threads of 16 walkers, 480 us with one wavefront; the spread search's evaluations: 38 to 17 us at
// 1024 walkers, 43 to 29 us at 3001; a batch of 64 mixed events: 1290 to 769 us).  The shape follows from
// the population alone, so an event has the same bits however it is run.
struct BranchShape {
    int wpt, threads;
};
constexpr BranchShape kBranchShapes[] = {{1, 64}, {1, 256}, {4, 256}, {4, 1024}, {kBranchWPT, kBranchThreads}};
constexpr int kBranchShapeCount = 5;
__host__ __device__ constexpr int branch_shape(int n)
{
    int i = 0;
    while (i < kBranchShapeCount - 1 && n > kBranchShapes[i].wpt * kBranchShapes[i].threads) ++i;
    return i;
}

// Walker l = threadIdx.x * WPT + q.  The weights w_l of the current
// Delta live in LDS (padded rows against bank conflicts), the branching
// words xi in registers, the residues too unless a thread has many walkers.
template <int WPT, int THREADS>
struct BranchShared {
    double dred[2][THREADS / 64];
    int ired[2][THREADS / 64];
    int scan[THREADS];
    int scan2[THREADS];
    double sw[THREADS * (WPT + 1)];
};

// Reduction over the branching workgroup with one barrier: each wavefront
// reduces in registers and publishes one partial, then every thread combines
// the partials.  Consecutive reductions alternate between two slot sets (par),
// so a reduction never overwrites partials that the previous one may still be
// reading; min, max and integer sums are exact in any order.
template <int WAVES, typename T, typename Op>
__device__ __forceinline__ T branch_reduce(T v, T (*slots)[WAVES], int &par, Op op)
{
    v = wave_reduce(v, op);
    if constexpr (WAVES == 1) return v;
    T *sl = slots[par];
    par ^= 1;
    if ((threadIdx.x & 63) == 0) sl[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = sl[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) r = op(r, sl[w]);
    return r;
}

// The fixed Delta search of one problem spread over many workgroups (64 walkers,
// an event: 480 us in one workgroup, 110 us of kernels spread):
// each round evaluates, in parallel, every Delta the search could visit next
// (the bracketing powers d0 2^j; then kTreeLevels levels of the bisection
// tree, each node's Delta derived from the round's bracket by the search's own
// sequence of square roots, so bit for bit the same values), and the last
// workgroup's walk applies the search's decisions to the results.  Zero counts do not
// depend on where inside the count-n interval of y an evaluation lands, so the
// walk takes exactly the decisions of the one-workgroup search.
constexpr int kTreeNear = 16;    // first bracketing round: d0 2^j, |j| <= kTreeNear
constexpr int kTreeFar = 200;    // the search's limit on halvings or doublings
constexpr int kTreeLevels = 8;   // bisection levels per round
constexpr int kBisections = 30;

struct BranchTree {
    double d0, lo, hi;
    double yhi, dhi;  // a y with sum m = N_w at Delta = dhi (the bracket's upper end), 0 if none
    int zt, degenerate;
    int ok;           // the bracket was found
    int dir;          // after the first round: 0 bracket found, -1 keep halving, +1 keep doubling
    unsigned int done;  // workgroups of the round that have finished (0 between rounds)
    int z[kTreeFar + (1 << kTreeLevels)];     // zero counts of the round's evaluations
    double y[kTreeFar + (1 << kTreeLevels)];  // their y (0 where none was found)
};

enum : int { kBranchSearch = 0, kBranchTreeEval = 1, kBranchTreeFinal = 2 };
enum : int { kRoundNear = 0, kRoundFar = 1, kRoundBisect = 2 };  // kRoundBisect + r: bisection round r

// Delta of bisection-tree node `node` (1: the root; children 2 node and
// 2 node + 1 take the lower and the upper half) inside the bracket [lo, hi].
__device__ __forceinline__ double tree_node_delta(double lo, double hi, int node)
{
    const int depth = 31 - __clz(node);
    for (int bit = depth - 1; bit >= 0; --bit) {
        const double mid = sqrt(lo * hi);
        if ((node >> bit) & 1) lo = mid;
        else hi = mid;
    }
    return sqrt(lo * hi);
}

// The workgroup's first THREADS threads solve the event (a launch for several
// shapes has more: their wavefronts leave at once).
template <int MODE, int WPT, int THREADS>
__device__ __forceinline__ void branch_block(const BranchArgs &a, BranchShared<WPT, THREADS> &sm, BranchTree *tree = nullptr,
                                             int round = 0)
{
    constexpr int ROW = WPT + 1;
    constexpr bool KEEP = WPT <= 4;  // residues in registers
    if ((int)threadIdx.x >= THREADS) return;
    auto dred = sm.dred;
    auto ired = sm.ired;
    int par = 0;
    int *scan = sm.scan;
    int *scan2 = sm.scan2;
    double *sw = sm.sw;
    const int n = a.n;
    const int l0 = threadIdx.x * WPT;
    const int nown = max(0, min(WPT, n - l0));
    double *myw = sw + threadIdx.x * ROW;
    uint32_t xw[WPT];
    int m[WPT];
    double kept[KEEP ? WPT : 1];
    auto read_chi2 = [&](int q) -> double {
        const double v = a.chi2[min(l0 + q, n - 1)];
        return (v == v) ? v : INFINITY;
    };
    if constexpr (KEEP) {
#pragma unroll
        for (int q = 0; q < WPT; ++q) kept[q] = read_chi2(q);
    }
    auto chi2_of = [&](int q) -> double {
        if constexpr (KEEP) return kept[q];
        else return read_chi2(q);
    };
    double cmin = INFINITY, cmax = -INFINITY;
#pragma unroll
    for (int q = 0; q < WPT; ++q) {
        uint32_t x0, x1, x2, x3;
        philox10((uint32_t)min(l0 + q, n - 1), a.event, 0u, kStreamBranch, a.key0, a.key1, x0, x1, x2, x3);
        xw[q] = x0;
        m[q] = 1;
        if (q < nown) {
            const double c = chi2_of(q);
            cmin = fmin(cmin, c);
            cmax = fmax(cmax, c);
        }
    }
    cmin = branch_reduce(cmin, dred, par, OpMin());
    cmax = branch_reduce(cmax, dred, par, OpMax());
#define XI(q) u01(xw[q])

    // For Delta, finds a y with sum m = n (then P = chi^2_min + ln(y)/Delta lies
    // between the n-th and (n+1)-th thresholds): bracket, then alternate secant
    // and bisection steps on the step function count(y).  Returns the zero
    // count at that y; *found = 0 on a tie.  One call site each for the
    // evaluation and the count keeps the kernel small.
    // guess > 0: a y expected near the answer (from the previous Delta); the
    // search then starts from [guess / 2, 2 guess] inside the full range.
    auto eval = [&](double delta, double guess, double *yout, int *found) __attribute__((always_inline)) -> int {
        double lo = INFINITY, hi = 0.0;
#pragma unroll KEEP ? WPT : 1
        for (int q = 0; q < WPT; ++q) myw[q] = (q < nown) ? exp(-(chi2_of(q) - cmin) * delta) : 0.0;
#pragma unroll
        for (int q = 0; q < WPT; ++q) {
            const double w = myw[q];
            if (q < nown && w > 0.0) {
                // walker q reaches m = 1 at y = (1 - xi) / w
                const double y1 = (1.0 - XI(q)) / w;
                lo = fmin(lo, y1);
                hi = fmax(hi, y1);
            }
        }
        lo = 0.5 * branch_reduce(lo, dred, par, OpMin());
        hi = 2.0 * branch_reduce(hi, dred, par, OpMax());
        const double lo0 = lo;  // count(lo0) = 0: no walker has reached m = 1
        if (guess > lo && guess < hi) {
            lo = fmax(lo, 0.5 * guess);
            hi = fmin(hi, 2.0 * guess);
        }
        // stage 0: count(hi), doubling hi until it reaches n; stage 1: count(lo),
        // lowered towards lo0 while it is not below n; stage 2: secant /
        // bisection inside [lo, hi].  Any y with count n gives the same result.
        int stage = 0, it = 0, clo = 0, chi = 0, zlast = 0;
        int side = 0, same = 0;  // the end the last interior step moved, and whether it repeated
        double y = hi, res = hi;
        *found = 0;
        for (;;) {
            int cnt = 0, zz = 0;
#pragma unroll
            for (int q = 0; q < WPT; ++q) {
                const int mq = (q < nown) ? branch_m(XI(q), myw[q], y, n) : 1;
                cnt += (q < nown) ? mq : 0;
                zz += (mq == 0);
            }
            cnt = branch_reduce(cnt, ired, par, OpSum());
            if (cnt == n) {
                res = y;
                zlast = zz;
                *found = 1;
                break;
            }
            if (stage == 0) {
                if (cnt < n) {
                    if (++it >= 64) break;
                    lo = hi;
                    hi = 2.0 * hi;
                    y = hi;
                    continue;
                }
                chi = cnt;
                res = hi;
                zlast = zz;
                stage = 1;
                it = 0;
                y = lo;
                continue;
            }
            if (stage == 1) {
                if (cnt >= n) {
                    if (lo > lo0) {
                        // started above the answer: this end becomes the upper one
                        hi = lo;
                        chi = cnt;
                        res = lo;
                        zlast = zz;
                        lo = fmax(lo0, 0.25 * lo);
                        y = lo;
                        if (++it > 400) break;
                        continue;
                    }
                    break;  // nothing strictly below n at the low end: tie
                }
                clo = cnt;
                stage = 2;
            } else if (cnt < n) {
                lo = y;
                clo = cnt;
                same = side == -1;
                side = -1;
            } else {
                hi = y;
                chi = cnt;
                res = y;
                zlast = zz;
                same = side == 1;
                side = 1;
            }
            if (++it > 400) break;
            double mid;
            if (hi > 4.0 * lo && lo > 0.0) {
                mid = sqrt(lo * hi);
            } else if (!same) {
                // secant step on the nearly linear count(y); a bisection
                // follows whenever one end moved twice in a row
                const double f = ((double)n + 0.5 - (double)clo) / (double)(chi - clo);
                mid = lo + (hi - lo) * f;
                if (!(mid > lo && mid < hi)) mid = 0.5 * (lo + hi);
            } else {
                mid = 0.5 * (lo + hi);
            }
            if (!(mid > lo && mid < hi)) break;
            y = mid;
        }
        *yout = res;
        return branch_reduce(zlast, ired, par, OpSum());
    };

    // adaptive branching (Sec. 2.5, last paragraph): fraction and imprint
    // strength scaled by the population mean of the running acceptance rate
    double fraction = a.fraction, t_eff = a.imprint_t;
    if (a.adaptive) {
        double rs = 0.0;
        for (int q = 0; q < nown; ++q) rs += a.rate[l0 + q];
        const double mean = branch_reduce(rs, dred, par, OpSum()) / (double)n;
        fraction *= mean;
        t_eff *= mean;
    }
    if (MODE != kBranchTreeEval && threadIdx.x == 0 && a.t_eff) *a.t_eff = t_eff;
    const int zt = (int)floor(fraction * (double)n + 0.5);
    int status = 0, z = 0;
    double delta = 0.0, pr = 0.0, gap = INFINITY, bracket = INFINITY;
    const bool degenerate = zt <= 0 || zt >= n || !(cmax > cmin) || !isfinite(cmax - cmin);
    if constexpr (MODE == kBranchTreeEval) {
        const double d0 = 1.0 / (cmax - cmin);
        if (round == kRoundNear && blockIdx.x == 0 && threadIdx.x == 0) {
            tree->d0 = d0;
            tree->zt = zt;
            tree->degenerate = degenerate ? 1 : 0;
        }
        if (degenerate) return;
        double dl;
        int slot;
        if (round == kRoundNear) {
            slot = blockIdx.x;
            dl = ldexp(d0, (int)blockIdx.x - kTreeNear);
        } else if (round == kRoundFar) {
            if (tree->dir == 0) return;
            slot = blockIdx.x;
            dl = ldexp(d0, tree->dir * (kTreeNear + 1 + (int)blockIdx.x));
        } else {
            if (!tree->ok) return;
            slot = blockIdx.x + 1;
            dl = tree_node_delta(tree->lo, tree->hi, slot);
        }
        // the y search starts from the bracket's upper end carried to this
        // Delta, as the one-workgroup search carries its last answer
        const double guess = (round >= kRoundBisect && tree->yhi > 0.0) ? exp(log(tree->yhi) * (dl / tree->dhi)) : 0.0;
        double Yd;
        int fd;
        const int zc = eval(dl, guess, &Yd, &fd);
        if (threadIdx.x == 0) {
            tree->z[slot] = zc;
            tree->y[slot] = fd ? Yd : 0.0;
        }
        return;
    }
    if (degenerate) {
        status = 1;
    } else {
        // the smallest Delta whose zero count reaches zt, from a fixed search:
        // start at 1/(max - min), halve or double to bracket, 30 bisections in
        // log Delta, then the upper end
        const double d0 = 1.0 / (cmax - cmin);
        double lo = 0.0, hi = 0.0, dcur = d0, Y = 0.0, ylast = 0.0, dlast = 0.0;
        int phase = 0, it = 0, fnd = 0, ok = 1;
        if constexpr (MODE == kBranchTreeFinal) {
            // the tree's bracket after the last bisection; the upper end, as the
            // one-workgroup search ends
            ok = tree->ok;
            if (ok) {
                lo = tree->lo;
                hi = tree->hi;
                const double guess = tree->yhi > 0.0 ? exp(log(tree->yhi) * (hi / tree->dhi)) : 0.0;
                z = eval(hi, guess, &Y, &fnd);
            }
        }
        for (; MODE == kBranchSearch;) {
            // y of the last solved Delta carried to this one: P = cmin + ln(y) / Delta
            const double guess = (ylast > 0.0) ? exp(log(ylast) * (dcur / dlast)) : 0.0;
            const int zc = eval(dcur, guess, &Y, &fnd);
            if (fnd) {
                ylast = Y;
                dlast = dcur;
            }
            if (phase == 0) {
                if (zc >= zt) {
                    hi = d0;
                    lo = 0.5 * d0;
                    phase = 1;
                    dcur = lo;
                } else {
                    lo = d0;
                    hi = 2.0 * d0;
                    phase = 2;
                    dcur = hi;
                }
            } else if (phase == 1) {
                if (zc >= zt) {
                    hi = lo;
                    lo = 0.5 * lo;
                    if (++it >= 200) {
                        ok = 0;
                        break;
                    }
                    dcur = lo;
                } else {
                    phase = 3;
                    it = 0;
                    dcur = sqrt(lo * hi);
                }
            } else if (phase == 2) {
                if (zc < zt) {
                    lo = hi;
                    hi = 2.0 * hi;
                    if (++it >= 200) {
                        ok = 0;
                        break;
                    }
                    dcur = hi;
                } else {
                    phase = 3;
                    it = 0;
                    dcur = sqrt(lo * hi);
                }
            } else if (phase == 3) {
                if (zc >= zt) hi = dcur; else lo = dcur;
                if (++it == 30) {
                    phase = 4;
                    dcur = hi;
                } else {
                    dcur = sqrt(lo * hi);
                }
            } else {
                z = zc;
                break;
            }
            __syncthreads();  // the weights in LDS are rewritten by the next evaluation
        }
        if (ok) {
            delta = hi;
#pragma unroll
            for (int q = 0; q < WPT; ++q) m[q] = (q < nown) ? branch_m(XI(q), myw[q], Y, n) : 0;
            // P_r: midpoint of the n-th and (n+1)-th smallest thresholds,
            // max_l theta_{l, m_l} and min_l theta_{l, m_l + 1}
            double thn = -INFINITY, thn1 = INFINITY;
#pragma unroll
            for (int q = 0; q < WPT; ++q) {
                if (q < nown) {
                    const double c = chi2_of(q);
                    if (m[q] >= 1) thn = fmax(thn, c + log((double)m[q] - XI(q)) / delta);
                    thn1 = fmin(thn1, c + log((double)(m[q] + 1) - XI(q)) / delta);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            thn = branch_reduce(thn, dred, par, OpMax());
            thn1 = branch_reduce(thn1, dred, par, OpMin());
            pr = 0.5 * (thn + thn1);
            // margins: the gap between those two thresholds relative to the
            // larger of their magnitudes and 1/Delta (small by construction: the
            // search ends just above the crossing that moves the zero count),
            // and the final bracket's relative width, within which that
            // crossing lies below Delta
            gap = (thn1 - thn) / fmax(fmax(fabs(thn), fabs(thn1)), 1.0 / delta);
            bracket = (hi - lo) / hi;
            status = (!fnd || thn == thn1) ? 2 : 0;
        } else {
            status = 1;
        }
        if (status != 0) {
#pragma unroll
            for (int q = 0; q < WPT; ++q) m[q] = 1;
        }
    }
    // pairing: zero-multiplier walkers in ascending order against donors in
    // ascending order, donor l repeated m_l - 1 times
    int nz = 0, nd = 0;
#pragma unroll
    for (int q = 0; q < WPT; ++q) {
        if (q < nown) {
            nz += (m[q] == 0);
            nd += max(m[q] - 1, 0);
        }
    }
    scan[threadIdx.x] = nz;
    scan2[threadIdx.x] = nd;
    __syncthreads();
    for (int off = 1; off < THREADS; off <<= 1) {
        const int v1 = (int)threadIdx.x >= off ? scan[threadIdx.x - off] : 0;
        const int v2 = (int)threadIdx.x >= off ? scan2[threadIdx.x - off] : 0;
        __syncthreads();
        scan[threadIdx.x] += v1;
        scan2[threadIdx.x] += v2;
        __syncthreads();
    }
    int zpos = scan[threadIdx.x] - nz, dpos = scan2[threadIdx.x] - nd;
    const int total_z = scan[THREADS - 1], total_d = scan2[THREADS - 1];
    const bool consistent = total_z == total_d;
#pragma unroll
    for (int q = 0; q < WPT; ++q) {
        if (q >= nown) continue;
        const int l = l0 + q;
        const int mq = consistent ? m[q] : 1;
        a.m[l] = mq;
        if (a.ev_m) a.ev_m[(size_t)a.event * n + l] = mq;
        if (!consistent) continue;
        if (mq == 0) a.targets[zpos++] = l;
        for (int cc = 1; cc < mq; ++cc) a.donors[dpos++] = l;
    }
    if (threadIdx.x == 0) {
        *a.npairs = (status == 0 && consistent) ? total_z : 0;
        a.ev_delta[a.event] = delta;
        a.ev_pr[a.event] = pr;
        a.ev_z[a.event] = z;
        a.ev_status[a.event] = (status == 0 && !consistent) ? 3 : status;
        a.ev_gap[a.event] = gap;
        a.ev_bracket[a.event] = bracket;
    }
#undef XI
}

// many problems: workgroup b solves the branching event of problem b
__global__ __launch_bounds__(kBranchThreads) void k_branch_batched(const BranchArgs *__restrict__ jobs)
{
    __shared__ BranchShared<kBranchWPT, kBranchThreads> sm;  // the largest shape's
    const BranchArgs a = jobs[blockIdx.x];
    auto solve = [&](auto shape) __attribute__((always_inline)) {
        constexpr BranchShape S = kBranchShapes[decltype(shape)::value];
        branch_block<kBranchSearch, S.wpt, S.threads>(a, reinterpret_cast<BranchShared<S.wpt, S.threads> &>(sm));
    };
    switch (branch_shape(a.n)) {
        case 0: solve(std::integral_constant<int, 0>{}); break;
        case 1: solve(std::integral_constant<int, 1>{}); break;
        case 2: solve(std::integral_constant<int, 2>{}); break;
        case 3: solve(std::integral_constant<int, 3>{}); break;
        default: solve(std::integral_constant<int, 4>{});
    }
}

// The search's decisions over one round's results (one thread).
__device__ __forceinline__ void branch_walk(BranchTree *t, int round, int levels)
{
    if (t->degenerate) return;
    const int zt = t->zt;
    const double d0 = t->d0;
    if (round == kRoundNear) {
        // z[kTreeNear + j] is the zero count at d0 2^j; halve while the count
        // at d0 reaches zt, else double
        t->ok = 0;
        const int *z = t->z + kTreeNear;
        const double *y = t->y + kTreeNear;
        if (z[0] >= zt) {
            for (int k = 1; k <= kTreeNear; ++k) {
                if (z[-k] < zt) {
                    t->lo = ldexp(d0, -k);
                    t->hi = ldexp(d0, 1 - k);
                    t->yhi = y[1 - k];
                    t->dhi = t->hi;
                    t->ok = 1;
                    t->dir = 0;
                    return;
                }
            }
            t->dir = -1;
            t->yhi = y[-kTreeNear];  // the upper end if the next round finds the crossing first
            t->dhi = ldexp(d0, -kTreeNear);
        } else {
            for (int k = 1; k <= kTreeNear; ++k) {
                if (z[k] >= zt) {
                    t->lo = ldexp(d0, k - 1);
                    t->hi = ldexp(d0, k);
                    t->yhi = y[k];
                    t->dhi = t->hi;
                    t->ok = 1;
                    t->dir = 0;
                    return;
                }
            }
            t->dir = 1;
        }
        return;
    }
    if (round == kRoundFar) {
        if (t->dir == 0) return;
        // z[k - kTreeNear - 1] at d0 2^(dir k); no crossing up to kTreeFar: the
        // search gives up (ok stays 0)
        for (int k = kTreeNear + 1; k <= kTreeFar; ++k) {
            const int zc = t->z[k - kTreeNear - 1];
            if (t->dir < 0 ? zc < zt : zc >= zt) {
                t->lo = t->dir < 0 ? ldexp(d0, -k) : ldexp(d0, k - 1);
                t->hi = t->dir < 0 ? ldexp(d0, 1 - k) : ldexp(d0, k);
                if (t->dir > 0) {
                    t->yhi = t->y[k - kTreeNear - 1];
                    t->dhi = t->hi;
                } else if (k > kTreeNear + 1) {
                    t->yhi = t->y[k - kTreeNear - 2];
                    t->dhi = t->hi;
                }
                t->ok = 1;
                return;
            }
        }
        return;
    }
    if (!t->ok) return;
    double lo = t->lo, hi = t->hi;
    int node = 1;
    for (int l = 0; l < levels; ++l) {
        const double mid = sqrt(lo * hi);
        if (t->z[node] >= zt) {
            hi = mid;
            t->yhi = t->y[node];
            t->dhi = mid;
            node = 2 * node;
        } else {
            lo = mid;
            node = 2 * node + 1;
        }
    }
    t->lo = lo;
    t->hi = hi;
}

// One round of the parallel Delta search: workgroup b evaluates the zero
// count at the round's b-th Delta.
template <int SHAPE>
__global__ __launch_bounds__(kBranchShapes[SHAPE].threads) void k_branch_tree(BranchArgs a, BranchTree *t, int round, int levels)
{
    if (round == kRoundFar && (t->degenerate || t->dir == 0)) return;
    if (round >= kRoundBisect && (t->degenerate || !t->ok)) return;
    constexpr BranchShape S = kBranchShapes[SHAPE];
    __shared__ BranchShared<S.wpt, S.threads> sm;
    branch_block<kBranchTreeEval, S.wpt, S.threads>(a, sm, t, round);
    // the last workgroup to finish applies the search's decisions (a launch of
    // its own took 5 us and a gap, six times an event)
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&t->done, 1u) == gridDim.x - 1) {
            __threadfence();
            branch_walk(t, round, levels);
            t->done = 0;
        }
    }
}

// The event itself at the tree's final Delta: multipliers, P_r, margins,
// pairing and the event log, as the one-workgroup kernel ends.
template <int SHAPE>
__global__ __launch_bounds__(kBranchShapes[SHAPE].threads) void k_branch_final(BranchArgs a, BranchTree *t)
{
    constexpr BranchShape S = kBranchShapes[SHAPE];
    __shared__ BranchShared<S.wpt, S.threads> sm;
    branch_block<kBranchTreeFinal, S.wpt, S.threads>(a, sm, t);
}

// --------------------------------------------------------------------------
// Outputs (Eq. residue-average over the walkers; chi^2 histogram)
// --------------------------------------------------------------------------
// Ensemble mean, bound by reading the spectra once: a workgroup takes kMeanBins
// bins (256-byte row segments) of up to kMeanSpan walkers, kMeanRows of them
// side by side, each thread its walkers in ascending order, the row sums added
// pairwise through LDS.  Populations of more than kMeanSpan walkers leave one
// partial sum per span, so that all compute units read (one workgroup per bin
// tile took 50 us over 64 MiB: a quarter of the compute units), and a second
// launch adds them in order.
// 512 bins x 16384 walkers: 4.0 ms with one thread per bin, 12 us (5.6 TB/s) and 4 us
// for the second launch now.
constexpr int kMeanBins = 32, kMeanRows = 32, kMeanSpan = 512;

int mean_spans(int n_walkers) { return (n_walkers + kMeanSpan - 1) / kMeanSpan; }

__global__ __launch_bounds__(kMeanBins * kMeanRows) void k_mean_spectrum(int n_walkers, int n_omega, const double *b,
                                                                         const double *gsc, double *out)
{
    __shared__ double part[kMeanRows][kMeanBins];
    const int c = threadIdx.x % kMeanBins, r = threadIdx.x / kMeanBins;
    const int j = blockIdx.x * kMeanBins + c;
    const int l0 = blockIdx.y * kMeanSpan, l1 = min(l0 + kMeanSpan, n_walkers);
    double s = 0.0;
    if (j < n_omega) {
#pragma unroll 8
        for (int l = l0 + r; l < l1; l += kMeanRows) s = fma(gsc[l], b[(size_t)l * n_omega + j], s);
    }
    part[r][c] = s;
    for (int h = kMeanRows / 2; h >= 1; h >>= 1) {
        __syncthreads();
        if (r < h) part[r][c] += part[r + h][c];
    }
    if (r == 0 && j < n_omega)
        out[(size_t)blockIdx.y * n_omega + j] = gridDim.y > 1 ? part[0][c] : part[0][c] / (double)n_walkers;
}

__global__ void k_mean_sum(int n_walkers, int n_omega, int spans, const double *part, double *out)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_omega) return;
    double s = part[j];
#pragma unroll 8
    for (int i = 1; i < spans; ++i) s += part[(size_t)i * n_omega + j];
    out[j] = s / (double)n_walkers;
}

// part: [mean_spans(n_walkers)][n_omega], may not overlap out
void launch_mean_spectrum(int n_walkers, int n_omega, const double *b, const double *gsc, double *part, double *out,
                          hipStream_t stream)
{
    const int spans = mean_spans(n_walkers);
    hipLaunchKernelGGL(k_mean_spectrum, dim3((unsigned)((n_omega + kMeanBins - 1) / kMeanBins), (unsigned)spans),
                       dim3(kMeanBins * kMeanRows), 0, stream, n_walkers, n_omega, b, gsc, spans > 1 ? part : out);
    if (spans > 1)
        hipLaunchKernelGGL(k_mean_sum, dim3((unsigned)((n_omega + 255) / 256)), dim3(256), 0, stream, n_walkers,
                           n_omega, spans, (const double *)part, out);
}

// Self-cooling temperature of block b (Sec. 2.4; reading: boil at the mean
// residue, a linear ramp from the mean to the minimum over `cool` blocks, then
// freeze at min / (1 + j)); one thread sums the residues in walker order (the
// workgroup stages them through LDS in chunks), and the block's sweeps
// [k0, k1) receive the temperature.
constexpr int kSelfCoolChunk = 4096;

__global__ void k_self_cool(const double *chi2, int n, int b, int boil, int cool, double *Tabs, int k0, int k1)
{
    __shared__ double Tb;
    __shared__ double buf[kSelfCoolChunk];
    double sum = 0.0, mn = chi2[0];
    for (int base = 0; base < n; base += kSelfCoolChunk) {
        const int cnt = min(kSelfCoolChunk, n - base);
        __syncthreads();  // the previous chunk has been consumed
        for (int i = (int)threadIdx.x; i < cnt; i += (int)blockDim.x) buf[i] = chi2[base + i];
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll 8
            for (int i = 0; i < cnt; ++i) {
                const double v = buf[i];
                sum += v;
                if (v < mn) mn = v;
            }
        }
    }
    if (threadIdx.x == 0) {
        const double mean = sum / (double)n;
        double T;
        if (b < boil) {
            T = mean;
        } else if (b < boil + cool) {
            const double x = (double)(b - boil + 1) / (double)cool;
            T = (1.0 - x) * mean + x * mn;
        } else {
            T = mn / (double)(1 + (b - boil - cool + 1));
        }
        Tb = T;
    }
    __syncthreads();
    for (int k = k0 + (int)threadIdx.x; k < k1; k += (int)blockDim.x) Tabs[k] = Tb;
}

constexpr int kHistMaxBins = 4096, kHistThreads = 256, kMinMaxThreads = 1024;

// Clears n words with vector stores (a kernel node, unlike a memset, is safe
// to record into a captured graph).
__global__ void k_zero_u64(int n, unsigned long long *v)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) v[i] = 0ull;
}

// Smallest and largest of n values, one workgroup (16384 values: 28 us with 256
// threads, 9 to 12 us with 1024; latency, four values in flight per thread).
__global__ __launch_bounds__(kMinMaxThreads) void k_minmax(int n, const double *v, double *out)
{
    __shared__ double red[kMinMaxThreads / 64];
    double lo = INFINITY, hi = -INFINITY;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        lo = fmin(lo, v[i]);
        hi = fmax(hi, v[i]);
    }
    lo = block_reduce(lo, red, OpMin());
    hi = block_reduce(hi, red, OpMax());
    if (threadIdx.x == 0) {
        out[0] = lo;
        out[1] = hi;
    }
}

// Histogram of log10 chi^2: counts first in the workgroup's LDS, so that the
// few bins of a population's residues meet in LDS rather than in one memory
// word (16384 residues in 64 bins: 43 us with one global atomic per residue,
// 4 us now).
__global__ __launch_bounds__(kHistThreads) void k_chi2_hist(int n, const double *chi2, int n_bins, double lo, double hi,
                                                           const double *range, unsigned long long *counts)
{
    __shared__ unsigned int local[kHistMaxBins];
    for (int i = threadIdx.x; i < n_bins; i += blockDim.x) local[i] = 0u;
    __syncthreads();
    if (range) {
        if (lo != lo) lo = log10(range[0]);
        if (hi != hi) hi = log10(range[1]);
    }
    const double width = hi - lo;
    for (int l = blockIdx.x * blockDim.x + threadIdx.x; l < n; l += gridDim.x * blockDim.x) {
        const double v = log10(chi2[l]);
        int bin = (width > 0.0) ? (int)floor((v - lo) / width * (double)n_bins) : 0;
        if (!(v == v)) bin = 0;
        bin = max(0, min(n_bins - 1, bin));
        atomicAdd(local + bin, 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_bins; i += blockDim.x)
        if (local[i]) atomicAdd(counts + i, (unsigned long long)local[i]);
}

// Clears the counts, finds the range where it is asked for (into range) and
// counts; range: two doubles, counts: n_bins words on the device.
hipError_t launch_chi2_hist(int n, const double *chi2, int n_bins, double lo, double hi, double *range,
                            unsigned long long *counts, hipStream_t stream)
{
    hipLaunchKernelGGL(k_zero_u64, dim3((n_bins + kThreads - 1) / kThreads), dim3(kThreads), 0, stream, n_bins, counts);
    const bool need_range = (lo != lo) || (hi != hi);
    if (need_range) hipLaunchKernelGGL(k_minmax, dim3(1), dim3(kMinMaxThreads), 0, stream, n, chi2, range);
    const int blocks = std::min(64, (n + kHistThreads - 1) / kHistThreads);
    hipLaunchKernelGGL(k_chi2_hist, dim3(blocks), dim3(kHistThreads), 0, stream, n, chi2, n_bins, lo, hi,
                       need_range ? (const double *)range : nullptr, counts);
    return hipGetLastError();
}

// Scratch of the allocation-free histogram (sail_read_chi2_hist_noalloc):
// words [0, kScratchRangeWords) hold the ensemble range as two doubles
// (padded to 256 bytes), the next kNoAllocMaxBins words the counts.  Every
// device the library runs on holds one copy until the process ends.  In host
// code this name is only a stand-in for the symbol: kernels receive the
// address hipGetSymbolAddress returns for the current device.
constexpr int kNoAllocMaxBins = kHistMaxBins;
constexpr int kScratchRangeWords = 32;
static __device__ __align__(256) unsigned long long scratch[kScratchRangeWords + kNoAllocMaxBins];

// --------------------------------------------------------------------------
// Host side
// --------------------------------------------------------------------------
// Device memory.  Outside a region every buffer is its own hipMalloc.  A
// served job's problem is built inside a Region: a block of the server's
// device arena that its buffers are carved from (no hipMalloc / hipFree, which
// would synchronise the device while other jobs run); freeing such a buffer
// is a no-op and the block returns to the arena as a whole.
struct Region {
    char *base = nullptr;
    size_t size = 0, used = 0;
    bool holds(const void *q) const { return base && (const char *)q >= base && (const char *)q < base + size; }
};
thread_local Region *g_region = nullptr;

struct RegionScope {
    Region *saved;
    explicit RegionScope(Region *r) : saved(g_region) { g_region = r; }
    ~RegionScope() { g_region = saved; }
};

// Device memory: hipMalloc, or the caller's allocator (sail_set_allocator).
// Pointers made by a caller's allocator are recorded with it, so each is
// returned to the allocator that made it even after the hook changed.
struct Allocator {
    sail_alloc_fn alloc = nullptr;
    sail_free_fn release = nullptr;
    void *user = nullptr;
};
struct Hooked {
    size_t bytes;
    int device;
    Allocator by;
};
std::mutex g_alloc_mu;
Allocator g_alloc;
std::map<void *, Hooked> g_hooked;

hipError_t raw_alloc(void **p, size_t bytes)
{
    Allocator a;
    {
        std::lock_guard<std::mutex> lk(g_alloc_mu);
        a = g_alloc;
    }
    if (!a.alloc) return hipMalloc(p, bytes);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    void *q = a.alloc(bytes, dev, a.user);
    if (!q) return hipErrorOutOfMemory;
    if (reinterpret_cast<uintptr_t>(q) & 255u) {
        a.release(q, bytes, dev, a.user);
        return hipErrorInvalidValue;
    }
    {
        std::lock_guard<std::mutex> lk(g_alloc_mu);
        g_hooked[q] = Hooked{bytes, dev, a};
    }
    *p = q;
    return hipSuccess;
}

void raw_free(void *p)
{
    if (!p) return;
    Hooked h{};
    bool hooked = false;
    {
        std::lock_guard<std::mutex> lk(g_alloc_mu);
        auto it = g_hooked.find(p);
        if (it != g_hooked.end()) {
            h = it->second;
            hooked = true;
            g_hooked.erase(it);
        }
    }
    if (!hooked) {
        (void)hipFree(p);
        return;
    }
    // hipFree waits for the device; a caller's allocator may hand the block
    // out again at once, so the device finishes its work on it first
    (void)hipDeviceSynchronize();
    h.by.release(p, h.bytes, h.device, h.by.user);
}

template <typename T>
sail_status dalloc(T **p, size_t count)
{
    *p = nullptr;
    if (count == 0) count = 1;
    const size_t bytes = count * sizeof(T);
    if (g_region) {
        const size_t off = (g_region->used + 255) & ~(size_t)255;
        if (off + bytes > g_region->size) return fail(SAIL_ENOMEM, "job region exhausted");
        *p = (T *)(g_region->base + off);
        g_region->used = off + bytes;
        return SAIL_OK;
    }
    hipError_t e = raw_alloc((void **)p, bytes);
    if (e != hipSuccess) return fail(SAIL_ENOMEM, std::string("device allocation: ") + hipGetErrorString(e));
    return SAIL_OK;
}

template <typename T>
void dfree(T *&p)
{
    if (p && !(g_region && g_region->holds(p))) raw_free((void *)p);
    p = nullptr;
}

// Device address of `scratch` on each device, taken once per device with that
// device current (every device holds its own copy at its own address).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned long long *g_scratch_addr[kMaxDevices] = {};

sail_status scratch_of_device(int device, unsigned long long **out)
{
    if (device < 0 || device >= kMaxDevices) return fail(SAIL_EINVAL, "device ordinal out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(SAIL_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_addr[device] = (unsigned long long *)ptr;
    }
    *out = g_scratch_addr[device];
    return SAIL_OK;
}

int next_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

}  // namespace

struct sail_problem {
    int device = 0;
    int n_omega = 0, n_tau = 0, mode = 0;
    double dw = 0, tau0 = 0, dtau = 0, A = 0, B = 0, m0 = 0, m1 = 0;
    std::vector<double> omega, tau, F, w, cfac;
    // nominal lane layout (sail_layout)
    int tpl = 16, lanes = 1, ntau_pad = 16;
    int tpl_hint = 0;  // requested tau points per lane (0: automatic)
    // tables (device); E holds the exact kernel columns and the columns in the basis
    double *d_tab = nullptr, *d_E = nullptr;  // d_tab holds the other tables
    double *d_omega = nullptr, *d_wh = nullptr, *d_Phit = nullptr, *d_cfac = nullptr;
    // walker-independent residue tables of the sweep (FP64): (omega, D, V, 0) per
    // bin and the pair-sum table (G, H), with the constant C and the grid's omega_0, d_omega
    double *d_bin = nullptr, *d_GH = nullptr;
    double tC = 0.0, tw0 = 0.0, tdW = 0.0;
    // the basis: dimensions per chunk for either precision (dimension d lies in
    // chunk d mod 4, so the FP32 loop's shorter basis is a prefix of every
    // chunk), and a digest of its vectors, which checkpoints carry
    int dims64 = 1, dims32 = 1, echunk = 2;
    uint64_t basis_id = 0;
    void *d_col = nullptr;  // columns in the loop precision, [N_omega][4][chunk()]
    int layout_precision = -1;
    int dims(int precision_) const { return precision_ == SAIL_FP32 ? dims32 : dims64; }
    int chunk(int precision_) const
    {
        return precision_ == SAIL_FP32 ? chunk_stride<float>(dims32) : chunk_stride<double>(dims64);
    }
    int cols() const { return n_tau + 4 * echunk; }
    int phi_row() const { return 4 * chunk(precision); }  // stored coordinates per walker
    // walkers (device)
    int n_walkers = 0, precision = 0;
    uint64_t seed = 0;
    double chi2_unit = NAN;
    double *d_b = nullptr, *d_gsc = nullptr /* scales, then d_rate, then d_F */, *d_ginv = nullptr, *d_chi2 = nullptr, *d_rate = nullptr;
    void *d_phi = nullptr;  // [N_w][4][chunk()] in the loop precision
    double *d_F = nullptr;  // [read_rows][n_tau], filled when reconstructions are read
    int read_rows = 0;
    // One read-out at a time uses the buffers kept for them (d_F, d_tmp, d_part,
    // d_hist): read-outs by several threads, which buffers of their own let run
    // side by side, take turns.
    std::mutex read_mu;
    double *d_a0 = nullptr, *d_tmp = nullptr, *d_teff = nullptr;  // d_teff: imprint strength of the last event
    double *d_part = nullptr;               // partial sums of the averaged spectrum
    unsigned long long *d_hist = nullptr;   // counts of the residue histogram, kept from its first call
    int cap_hist = 0;
    int32_t *d_m = nullptr, *d_targets = nullptr, *d_donors = nullptr, *d_npairs = nullptr;
    BranchTree *d_tree = nullptr;  // state of the parallel Delta search
    // events
    int cap_events = 0, keep_m = 0;
    double *d_ev_delta = nullptr, *d_ev_pr = nullptr, *d_ev_gap = nullptr, *d_ev_bracket = nullptr;
    int32_t *d_ev_z = nullptr, *d_ev_status = nullptr, *d_ev_m = nullptr;
    // schedule
    double *d_Tabs = nullptr;
    int cap_T = 0;
    int self_T_k0 = 0, self_T_end = 0;  // self-cooling: the block whose temperature d_Tabs holds last
    std::vector<double> h_Tabs;  // what d_Tabs holds
    // watchdog (failure detection): snapshot of the walker state at the last
    // clean check, and the flag / sweep words the kernels update
    double watch_bound = 0.0;
    bool watch_active = false;  // set while sail_run_schedule runs with the watchdog on
    unsigned int *d_watch = nullptr;
    double *sn_b = nullptr, *sn_gsc = nullptr, *sn_ginv = nullptr, *sn_chi2 = nullptr, *sn_rate = nullptr;
    double *sn_phi = nullptr;  // the loop-precision phi as raw 8-byte words
    int watch_tripped = -1, watch_restored = -1;
    // per-block log: a ring of records and the walkers' drift at the last resync
    sail_block_record *d_blog = nullptr;
    double *d_drift = nullptr;
    int blog_cap = 0;
    int64_t blog_total = 0;
    // trace
    int tk0 = 0, tk1 = 0;
    double *tr_dchi2 = nullptr;
    uint8_t *tr_flags = nullptr;
    // timing
    int timing = 0;
    std::vector<hipEvent_t> ev_start, ev_stop;
    size_t ev_used = 0;
    // completion of the last enqueued anneal work (sail_read_events waits on it
    // from a private stream instead of synchronising the device)
    hipEvent_t done_ev = nullptr;
    hipStream_t read_stream = nullptr;

    void free_walkers()
    {
        dfree(d_b); dfree(d_phi); dfree(d_gsc); dfree(d_ginv); dfree(d_chi2);
        d_rate = d_F = nullptr;  // (parts of d_gsc)
        dfree(d_a0); dfree(d_tmp); dfree(d_teff); dfree(d_part); dfree(d_hist); dfree(d_m); dfree(d_targets); dfree(d_donors); dfree(d_npairs);
        dfree(d_tree);
        dfree(d_ev_delta); dfree(d_ev_pr); dfree(d_ev_z); dfree(d_ev_status); dfree(d_ev_m);
        dfree(d_ev_gap); dfree(d_ev_bracket);
        free_watch();
        free_block_log();
        cap_events = 0;
        cap_hist = 0;
        n_walkers = 0;
    }
    void free_block_log()
    {
        dfree(d_blog); dfree(d_drift);
        blog_cap = 0;
        blog_total = 0;
    }
    void free_watch()
    {
        dfree(d_watch); dfree(sn_b); dfree(sn_gsc); dfree(sn_ginv); dfree(sn_chi2); dfree(sn_rate); dfree(sn_phi);
        watch_bound = 0.0;
    }
    ~sail_problem()
    {
        (void)hipSetDevice(device);
        free_walkers();
        dfree(d_tab); dfree(d_E); dfree(d_Tabs); dfree(d_col);
        for (auto e : ev_start) (void)hipEventDestroy(e);
        for (auto e : ev_stop) (void)hipEventDestroy(e);
        if (done_ev) (void)hipEventDestroy(done_ev);
        if (read_stream) (void)hipStreamDestroy(read_stream);
    }
};

namespace {

bool finite_all(const double *v, int n)
{
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(v[i])) return false;
    return true;
}

bool uniform_grid(const double *v, int n, double *step)
{
    if (n < 2) {
        *step = 0.0;
        return true;
    }
    const double h = (v[n - 1] - v[0]) / (double)(n - 1);
    double scale = std::max(std::fabs(v[0]), std::fabs(v[n - 1]));
    for (int i = 0; i < n; ++i)
        if (std::fabs(v[i] - (v[0] + h * (double)i)) > 1e-12 * scale) return false;
    *step = h;
    return h > 0.0;
}

// Maximum-entropy start a_j ~ e^{-lambda omega_j} with sum a = A and
// sum a omega = B: Newton iteration on lambda for the tilted mean, kept inside
// a bracket that is halved whenever a Newton step would leave it.
sail_status start_spectrum(const std::vector<double> &om, double A, double B, std::vector<double> &a)
{
    const int n = (int)om.size();
    const double mu = B / A;
    auto moments = [&](double lam, double &mean, double &var) {
        const double ref = lam > 0.0 ? om[0] : om[n - 1];
        double s0 = 0, s1 = 0, s2 = 0;
        for (int j = 0; j < n; ++j) {
            const double e = std::exp(-lam * (om[j] - ref));
            s0 += e;
            s1 += e * om[j];
            s2 += e * om[j] * om[j];
        }
        mean = s1 / s0;
        var = s2 / s0 - mean * mean;
    };
    double lo = -1.0, hi = 1.0, mean, var;
    for (int it = 0; it < 4000; ++it) { moments(lo, mean, var); if (mean > mu) break; lo *= 2.0; }
    for (int it = 0; it < 4000; ++it) { moments(hi, mean, var); if (mean < mu) break; hi *= 2.0; }
    double lam = 0.0;
    moments(lam, mean, var);
    if (mean != mu) {
        lam = 0.5 * (lo + hi);
        for (int it = 0; it < 500; ++it) {
            moments(lam, mean, var);
            if (mean == mu) break;
            if (mean > mu) lo = lam; else hi = lam;
            // d mean / d lambda = -var
            double next = (var > 0.0) ? lam + (mean - mu) / var : 0.5 * (lo + hi);
            if (!(next > lo && next < hi)) next = 0.5 * (lo + hi);
            if (next == lam || hi - lo <= 4e-16 * std::max(std::fabs(lo), std::fabs(hi))) break;
            lam = next;
        }
    }
    const double ref = lam > 0.0 ? om[0] : om[n - 1];
    a.assign(n, 0.0);
    double s = 0.0;
    for (int j = 0; j < n; ++j) {
        a[j] = std::exp(-lam * (om[j] - ref));
        s += a[j];
    }
    for (int j = 0; j < n; ++j) a[j] = a[j] * (A / s);
    // two-parameter correction of both sums
    double s0 = 0, s1 = 0, s2 = 0;
    for (int j = 0; j < n; ++j) {
        s0 += a[j];
        s1 += a[j] * om[j];
        s2 += a[j] * om[j] * om[j];
    }
    const double e0 = A - s0, e1 = B - s1, det = s0 * s2 - s1 * s1;
    if (det > 0.0) {
        const double d0 = (e0 * s2 - e1 * s1) / det, d1 = (e1 * s0 - e0 * s1) / det;
        for (int j = 0; j < n; ++j) a[j] = a[j] + a[j] * (d0 + d1 * om[j]);
    }
    return SAIL_OK;
}

// Marks the end of the work just enqueued on `stream` for this problem.
sail_status mark_done(sail_problem *p, hipStream_t stream)
{
    if (!p->done_ev) SAIL_HIP(hipEventCreateWithFlags(&p->done_ev, hipEventDisableTiming));
    SAIL_HIP(hipEventRecord(p->done_ev, stream));
    return SAIL_OK;
}

sail_status ensure_events(sail_problem *p, int need, hipStream_t stream)
{
    if (need <= p->cap_events) return SAIL_OK;
    int cap = std::max(need, 2 * p->cap_events);
    double *nd = nullptr, *np = nullptr, *ng = nullptr, *nb = nullptr;
    int32_t *nz = nullptr, *ns = nullptr, *nm = nullptr;
    sail_status st;
    if ((st = dalloc(&nd, cap)) || (st = dalloc(&np, cap)) || (st = dalloc(&nz, cap)) || (st = dalloc(&ns, cap)) ||
        (st = dalloc(&ng, cap)) || (st = dalloc(&nb, cap))) {
        dfree(nd); dfree(np); dfree(nz); dfree(ns); dfree(ng); dfree(nb);
        return st;
    }
    if (p->keep_m && (st = dalloc(&nm, (size_t)cap * p->n_walkers))) {
        dfree(nd); dfree(np); dfree(nz); dfree(ns); dfree(ng); dfree(nb);
        return st;
    }
    SAIL_HIP(hipMemsetAsync(ns, 0xff, sizeof(int32_t) * cap, stream));
    if (p->cap_events > 0) {
        SAIL_HIP(hipMemcpyAsync(nd, p->d_ev_delta, sizeof(double) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipMemcpyAsync(np, p->d_ev_pr, sizeof(double) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipMemcpyAsync(nz, p->d_ev_z, sizeof(int32_t) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipMemcpyAsync(ns, p->d_ev_status, sizeof(int32_t) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipMemcpyAsync(ng, p->d_ev_gap, sizeof(double) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipMemcpyAsync(nb, p->d_ev_bracket, sizeof(double) * p->cap_events, hipMemcpyDeviceToDevice, stream));
        if (nm && p->d_ev_m)
            SAIL_HIP(hipMemcpyAsync(nm, p->d_ev_m, sizeof(int32_t) * p->cap_events * p->n_walkers, hipMemcpyDeviceToDevice, stream));
        SAIL_HIP(hipStreamSynchronize(stream));
    }
    dfree(p->d_ev_delta); dfree(p->d_ev_pr); dfree(p->d_ev_z); dfree(p->d_ev_status); dfree(p->d_ev_m);
    dfree(p->d_ev_gap); dfree(p->d_ev_bracket);
    p->d_ev_delta = nd; p->d_ev_pr = np; p->d_ev_z = nz; p->d_ev_status = ns; p->d_ev_m = nm;
    p->d_ev_gap = ng; p->d_ev_bracket = nb;
    p->cap_events = cap;
    return SAIL_OK;
}

ResyncArgs make_resync_args(const sail_problem *p, int renorm, const int32_t *list, const int32_t *list_count,
                            int n_items, const int32_t *donors, double imprint_t, double smooth = 0.0,
                            const double *imprint_t_dev = nullptr)
{
    ResyncArgs r;
    r.n_omega = p->n_omega;
    r.n_tau = p->n_tau;
    r.cols = p->cols();
    r.echunk = p->echunk;
    r.chunk = p->chunk(p->precision);
    r.omega = p->d_omega;
    r.E = p->d_E;
    r.wh = p->d_wh;
    r.Phit = p->d_Phit;
    r.b = p->d_b;
    r.gsc = p->d_gsc;
    r.ginv = p->d_ginv;
    r.phi = p->d_phi;
    r.chi2 = p->d_chi2;
    r.A = p->A;
    r.B = p->B;
    r.renorm = renorm;
    r.list = list;
    r.list_count = list_count;
    r.n_items = n_items;
    r.donors = donors;
    r.imprint_t = imprint_t;
    r.imprint_t_dev = imprint_t_dev;
    r.smooth = smooth;
    r.watch = nullptr;
    r.watch_bound = INFINITY;
    r.drift = nullptr;
    return r;
}

// Batched resyncs are launched per class of that LDS size: N_omega up to
// 256, 512, 1024, and beyond.
constexpr int kResyncClasses = 4;
int resync_class(int n_omega) { return n_omega <= 256 ? 0 : n_omega <= 512 ? 1 : n_omega <= 1024 ? 2 : 3; }
// Walkers per resync workgroup: 16 fill the matrix instructions' rows, where two
// such workgroups fit a compute unit and there are more than 8 walkers per compute
// unit (a resync with its launch, 16 against 8 walkers: 512 bins, 16384 walkers
// 133 and 168 us, 3000 walkers 48 and 62 us); else 8 (256 bins, 2048 walkers 38
// and 27 us; 1000 bins, 8000 walkers 210 and 212 us, and 8 take half the LDS).
int resync_wpb(int n_omega, size_t n_items) { return n_omega <= 512 && n_items > 8 * 256 ? 16 : 8; }
// its LDS: the walkers' spectra, then the per-wavefront residue partials
size_t resync_shmem(int n_omega, int wpb) { return sizeof(double) * wpb * (resync_stride(n_omega) + 4); }
int resync_blocks(int n_items, int wpb) { return (n_items + wpb - 1) / wpb; }
template <typename R>
void launch_resync_k(int wpb, int blocks, size_t shm, hipStream_t stream, const ResyncArgs &r)
{
    if (wpb == 16) hipLaunchKernelGGL((k_resync<R, 16>), dim3(blocks), dim3(kThreads), shm, stream, r);
    else hipLaunchKernelGGL((k_resync<R, 8>), dim3(blocks), dim3(kThreads), shm, stream, r);
}
template <typename R>
void launch_resync_k(int wpb, int blocks, size_t shm, hipStream_t stream, const ResyncArgs *r, const int *first, int n)
{
    if (wpb == 16) hipLaunchKernelGGL((k_resync_batched<R, 16>), dim3(blocks), dim3(kThreads), shm, stream, r, first, n);
    else hipLaunchKernelGGL((k_resync_batched<R, 8>), dim3(blocks), dim3(kThreads), shm, stream, r, first, n);
}

// LDS one workgroup may hold on gfx950 (the 160 KiB of a compute unit).
constexpr size_t kLdsBytes = 160 * 1024;

// The resync stages 8 spectra per workgroup at least, so N_omega is bounded by
// the LDS of one workgroup (N_omega <= 2556 on gfx950); a sweep needs its
// records only (its tables are read from memory where they do not fit).
sail_status check_lds(int n_omega, size_t limit = kLdsBytes)
{
    const size_t resync = resync_shmem(n_omega, 8);
    if (resync > limit)
        return fail(SAIL_EINVAL, "n_omega = " + std::to_string(n_omega) + " needs " + std::to_string(resync) +
                                     " bytes of LDS per workgroup; " + std::to_string(limit) + " are available");
    return SAIL_OK;
}

// Resync of n_items walkers (all, or the first *list_count of `list`),
// optionally after imprinting donors[i] into list[i].
sail_status launch_resync(sail_problem *p, int renorm, const int32_t *list, const int32_t *list_count, int n_items,
                          hipStream_t stream, const int32_t *donors = nullptr, double imprint_t = 0.0,
                          double smooth = 0.0, const double *imprint_t_dev = nullptr)
{
    ResyncArgs r = make_resync_args(p, renorm, list, list_count, n_items, donors, imprint_t, smooth, imprint_t_dev);
    if (p->watch_active) {
        // every resync checks chi^2; the plain renormalising one also the
        // drift (smoothing moves the first moment on purpose)
        r.watch = p->d_watch;
        r.watch_bound = (renorm && !donors && !(smooth > 0.0)) ? p->watch_bound : INFINITY;
    }
    if (p->d_drift && renorm && !list && !donors && !(smooth > 0.0)) r.drift = p->d_drift;
    const int wpb = resync_wpb(p->n_omega, n_items), blocks = resync_blocks(n_items, wpb);
    const size_t shmem = resync_shmem(p->n_omega, wpb);
    if (p->precision == SAIL_FP32) launch_resync_k<float>(wpb, blocks, shmem, stream, r);
    else launch_resync_k<double>(wpb, blocks, shmem, stream, r);
    SAIL_HIP(hipGetLastError());
    return SAIL_OK;
}

// One branching event of a single problem: a few rounds over many workgroups.
template <int SHAPE>
void launch_branch_tree(const BranchArgs &ba, BranchTree *t, hipStream_t stream)
{
    constexpr int T = kBranchShapes[SHAPE].threads;
    hipLaunchKernelGGL(k_branch_tree<SHAPE>, dim3(2 * kTreeNear + 1), dim3(T), 0, stream, ba, t, (int)kRoundNear, 0);
    hipLaunchKernelGGL(k_branch_tree<SHAPE>, dim3(kTreeFar - kTreeNear), dim3(T), 0, stream, ba, t, (int)kRoundFar, 0);
    for (int r = 0, done = 0; done < kBisections; ++r) {
        const int lv = std::min(kTreeLevels, kBisections - done);
        hipLaunchKernelGGL(k_branch_tree<SHAPE>, dim3((1 << lv) - 1), dim3(T), 0, stream, ba, t, kRoundBisect + r, lv);
        done += lv;
    }
    hipLaunchKernelGGL(k_branch_final<SHAPE>, dim3(1), dim3(T), 0, stream, ba, t);
}

sail_status launch_branch(sail_problem *p, const BranchArgs &ba, hipStream_t stream)
{
    const int shape = branch_shape(p->n_walkers);
    switch (shape) {
        case 0: launch_branch_tree<0>(ba, p->d_tree, stream); break;
        case 1: launch_branch_tree<1>(ba, p->d_tree, stream); break;
        case 2: launch_branch_tree<2>(ba, p->d_tree, stream); break;
        case 3: launch_branch_tree<3>(ba, p->d_tree, stream); break;
        default: launch_branch_tree<4>(ba, p->d_tree, stream);
    }
    SAIL_HIP(hipGetLastError());
    return SAIL_OK;
}

BranchArgs make_branch_args(const sail_problem *p, double fraction, int event, int adaptive = 0, double imprint_t = 0.0)
{
    BranchArgs ba;
    ba.n = p->n_walkers;
    ba.chi2 = p->d_chi2;
    ba.rate = p->d_rate;
    ba.adaptive = adaptive;
    ba.imprint_t = imprint_t;
    ba.t_eff = adaptive ? p->d_teff : nullptr;
    ba.key0 = (uint32_t)p->seed;
    ba.key1 = (uint32_t)(p->seed >> 32);
    ba.event = (uint32_t)event;
    ba.fraction = fraction;
    ba.m = p->d_m;
    ba.targets = p->d_targets;
    ba.donors = p->d_donors;
    ba.npairs = p->d_npairs;
    ba.ev_delta = p->d_ev_delta;
    ba.ev_pr = p->d_ev_pr;
    ba.ev_z = p->d_ev_z;
    ba.ev_status = p->d_ev_status;
    ba.ev_m = p->keep_m ? p->d_ev_m : nullptr;
    ba.ev_gap = p->d_ev_gap;
    ba.ev_bracket = p->d_ev_bracket;
    return ba;
}

struct SweepParams {
    double eps0, amp_p, amp_avg;
    int amp_m, walk_len;
};

int sweep_wg_sync()
{
    static const int v = [] {
        const char *env = std::getenv("SAIL_SWEEP_SYNC");
        return env ? std::atoi(env) : 0;
    }();
    return v;
}

// How a sweep is launched: split or not, lanes per walker, threads and walkers
// per workgroup, whether the columns and the walkers' spectra sit in LDS, and
// the LDS they take with the records.  The results have the same bits for any
// plan.
struct SweepPlan {
    bool split;
    int lanes, threads, walkers;
    int columns_lds, spectra_lds, tables_lds;
    int resident;  // split: bins of every spectrum in LDS
    size_t shm;
};

SweepArgs make_sweep_args(const sail_problem *p, int k0, int k1, const SweepParams &sp, const SweepPlan &plan)
{
    SweepArgs s;
    s.n_walkers = p->n_walkers;
    s.n_omega = p->n_omega;
    s.columns_lds = plan.columns_lds;
    s.tables_lds = plan.tables_lds;
    s.resident = plan.resident;
    s.lanes = plan.lanes;
    s.pairs = plan.threads / 128;
    s.k0 = k0;
    s.k1 = k1;
    s.key0 = (uint32_t)p->seed;
    s.key1 = (uint32_t)(p->seed >> 32);
    s.A = p->A;
    s.B = p->B;
    s.eps0 = sp.eps0;
    s.amp_p = sp.amp_p;
    s.amp_avg = sp.amp_avg;
    s.amp_m = sp.amp_m;
    s.col = p->d_col;
    s.phi = p->d_phi;
    s.bin = (const double4 *)p->d_bin;
    s.GH = (const double2 *)p->d_GH;
    s.C = p->tC;
    s.w0 = p->tw0;
    s.dW = p->tdW;
    s.b = p->d_b;
    s.gsc = p->d_gsc;
    s.ginv = p->d_ginv;
    s.chi2 = p->d_chi2;
    s.rate = p->d_rate;
    s.Tabs = p->d_Tabs;
    s.tk0 = p->tk0;
    s.tk1 = p->tk1;
    s.tr_dchi2 = p->tr_dchi2;
    s.tr_flags = p->tr_flags;
    s.wg_sync = sweep_wg_sync();
    // diagnostic: SAIL_EXACT_THRESHOLD=1 takes every decision with the FP64 log
    const char *ex = std::getenv("SAIL_EXACT_THRESHOLD");
    s.thr_tol = (ex && std::atoi(ex) != 0) ? INFINITY : kThrTol;
    s.walk_len = sp.walk_len;
    return s;
}

// The columns, then the spectra of the workgroup's walkers (if asked for), go
// to LDS if they fit in `budget` bytes beside the records.  A walk's kernels, and
// those of one wavefront, take both or neither.
SweepPlan plan_sweep(const sail_problem *p, bool split, int lanes, int threads, size_t budget, bool walk, bool spectra,
                     int walk_len)
{
    const int walkers = (split ? threads / 2 : threads) / lanes;
    SweepPlan s{split, lanes, threads, walkers, 0, 0, 0, 0,
                sizeof(double) * (!split ? (size_t)walkers * rec_stride(lanes, walk)
                                  : walk ? (size_t)walkers * walk_split_stride(walk_len)
                                         : (size_t)walkers * split_stride(lanes) + (size_t)walkers / (64 / lanes) * split_hits(lanes))};
    const size_t col = column_bytes(p->n_omega, p->chunk(p->precision),
                                    p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double));
    const size_t spec = sizeof(double) * (size_t)walkers * p->n_omega;
    // (a split walk: and the tables of the bins and their pairs)
    const size_t bins = (size_t)p->n_omega * sizeof(double4), tables = bins + (size_t)(2 * p->n_omega - 1) * sizeof(double2);
    const size_t all = !split || !walk ? spec : ((spec + 15) & ~(size_t)15) + tables;
    const bool fits = spectra && s.shm + col + all <= budget;
    if ((walk || !split) ? !fits : s.shm + col > budget) {
        s.tables_lds = s.shm + tables <= budget ? 2 : s.shm + bins <= budget ? 1 : 0;
        s.shm += s.tables_lds == 2 ? tables : s.tables_lds == 1 ? bins : 0;
        return s;
    }
    if (s.shm + col <= budget) {
        s.shm += col;
        s.columns_lds = 1;
        if (!(split && lanes == 4) && fits) {
            s.shm += all;
            s.spectra_lds = 1;
        }
        // Many walkers per compute unit: the spectra in flight outgrow the L2
        // caches (8 MB per 4 MB cache at 512 bins), and the sweep waits for the
        // memory behind them.  What LDS is left keeps the first bins of each
        // (512 bins, 16384 walkers: 14 % of them in FP64, 27 % in FP32; block
        // 22.9 to 20.6 ms and 22.9 to 18.7 ms).  Smaller workgroups mean
        // spectra that the caches hold, where the extra instructions lose 2 %
        // (24 FP64 jobs: 27.2 to 27.8 ms; band: 26.0 to 26.6 ms).
        if (split && lanes == 4 && threads == 2 * kSweepThreads) {
            const int slots = (int)((budget - s.shm) / (sizeof(double) * (size_t)walkers));
            s.resident = std::min(std::max(slots - 1, 0), p->n_omega);
            if (s.resident) s.shm += sizeof(double) * (size_t)walkers * (s.resident + 1);
        }
    }
    return s;
}

int sweep_blocks(const sail_problem *p, const SweepPlan &s) { return (p->n_walkers + s.walkers - 1) / s.walkers; }

bool sweep_traced(const sail_problem *p, int k0, int k1) { return p->tk1 > p->tk0 && k0 < p->tk1 && k1 > p->tk0; }

constexpr int kCUs = 256;

// The plan of a problem swept alone.  Workgroups are the smallest that leave at
// most one per compute unit, so that a small population spreads over the chip,
// each with as much LDS as its share of a compute unit.  In order of
// preference (times of one proposal of every walker):
//   split, 16 lanes a walker, spectra in LDS beside the columns, for up to 16
//     walkers per compute unit: 196 ns (64 bins, 64 walkers) and 215 ns (300
//     bins, 3000 walkers), against 207 and 220 ns in one wavefront (the next);
//   16 lanes in one wavefront, which stages its own proposals: its records take
//     two thirds of the LDS, so that larger spectra fit;
//   split, 16 lanes, spectra in memory: a batch's loads, stores and masks of
//     shared bins are paid once in 16 proposals: 215 ns (1000 bins, 1500
//     walkers), against 244 ns for four lanes;
//   split, four lanes a walker: 64 walkers per compute unit at a time, 360 ns
//     (512 bins, 16384 walkers); also where the columns fit beside these smaller
//     records only (900 bins, 3500 walkers: 246 against 253 ns).
SweepPlan plan_alone(const sail_problem *p, int mode, int walk_len)
{
    const size_t n = (size_t)p->n_walkers;
    const int wide = wide_basis(p->dims(p->precision)) ? 16 : 0;  // lanes a wide basis takes
    auto sized = [&](bool split, int lanes, bool spectra) {
        const int most = split ? 2 * kSweepThreads : kSweepThreads, per = split ? 2 * lanes : lanes;
        int threads = split ? 128 : 64;
        while (threads < most && n * per > (size_t)threads * kCUs) threads *= 2;
        const size_t blocks = (n * per + threads - 1) / threads;
        // (a split sweep's registers leave room for one workgroup of eight wavefronts)
        const size_t per_cu = split ? 1 : std::min<size_t>(std::max<size_t>((blocks + kCUs - 1) / kCUs, 1), 4);
        return plan_sweep(p, split, lanes, threads, kLdsBytes / per_cu, mode == kSweepWalk, spectra, walk_len);
    };
    if (mode == kSweepTraced) return sized(false, wide ? wide : 4, false);
    // Walks: split, 16 lanes a walker, everything in LDS, if it fits; else all in
    // one wavefront, 8 lanes a walker (256 bins, 1024 walkers, 4 steps: a block
    // 3.5 ms against 6.4 ms, and 9.3 ms with the tables in memory).
    if (mode == kSweepWalk) {
        const SweepPlan w = sized(true, 16, true);
        return w.spectra_lds ? w : sized(false, wide ? wide : 8, true);
    }
    if (n * 16 <= (size_t)kSweepThreads * kCUs) {
        const SweepPlan t = sized(true, 16, true);
        if (t.spectra_lds) return t;
        const SweepPlan u = sized(false, 16, true);
        if (u.spectra_lds) return u;
        if (t.columns_lds) return t;
    }
    const SweepPlan s = sized(false, 16, true);
    return s.spectra_lds ? s : sized(true, wide ? wide : 4, false);
}

template <typename R, int M, int G, bool LDSC, bool LDSB, int MODE>
void launch_sweep_k(const SweepArgs &a, int blocks, const SweepPlan &s, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sweep<R, M, G, LDSC, LDSB, MODE>), dim3(blocks), dim3(s.threads), s.shm, stream, a);
}

template <typename R, int M>
void launch_sweep_m(const SweepArgs &a, int blocks, const SweepPlan &s, int mode, hipStream_t stream)
{
    constexpr bool WIDE = wide_basis(M);
    const dim3 grid(blocks), thr(s.threads);
    if (mode == kSweepTraced) return launch_sweep_k<R, M, WIDE ? 16 : 4, false, false, kSweepTraced>(a, blocks, s, stream);
    if (mode == kSweepWalk) {
        if (s.split) hipLaunchKernelGGL((k_sweep_split16<R, M, true, true, kSweepWalk>), grid, thr, s.shm, stream, a);
        else if (s.spectra_lds) launch_sweep_k<R, M, WIDE ? 16 : 8, true, true, kSweepWalk>(a, blocks, s, stream);
        else launch_sweep_k<R, M, WIDE ? 16 : 8, false, false, kSweepWalk>(a, blocks, s, stream);
        return;
    }
    if (s.spectra_lds) {
        if (s.split) hipLaunchKernelGGL((k_sweep_split16<R, M, true, true, kSweepFast>), grid, thr, s.shm, stream, a);
        else launch_sweep_k<R, M, 16, true, true, kSweepFast>(a, blocks, s, stream);
        return;
    }
    // (spectra in memory: split; 16 lanes with the columns in LDS, or a wide basis)
    if (s.lanes == 16 && s.columns_lds) {
        hipLaunchKernelGGL((k_sweep_split16<R, M, true, false, kSweepFast>), grid, thr, s.shm, stream, a);
    } else if constexpr (WIDE) {
        hipLaunchKernelGGL((k_sweep_split16<R, M, false, false, kSweepFast>), grid, thr, s.shm, stream, a);
    } else if (s.resident) {
        hipLaunchKernelGGL((k_sweep_split<R, M, true, true>), grid, thr, s.shm, stream, a);
    } else if (s.columns_lds) {
        hipLaunchKernelGGL((k_sweep_split<R, M, true, false>), grid, thr, s.shm, stream, a);
    } else {
        hipLaunchKernelGGL((k_sweep_split<R, M, false, false>), grid, thr, s.shm, stream, a);
    }
}

// Calls f(R{}, std::integral_constant<int, M>{}) for the kernel of a basis class.
template <typename F>
void with_basis_class(int precision, int cls, F &&f)
{
#define SAIL_CASE(R, M) case M: f(R{}, std::integral_constant<int, M>{}); break;
    if (precision == SAIL_FP32) {
        switch (cls) {
            SAIL_CASE(float, 2) SAIL_CASE(float, 3) SAIL_CASE(float, 4) SAIL_CASE(float, 6) SAIL_CASE(float, 16)
            SAIL_CASE(float, 24)
        }
    } else {
        switch (cls) {
            SAIL_CASE(double, 2) SAIL_CASE(double, 4) SAIL_CASE(double, 6) SAIL_CASE(double, 8) SAIL_CASE(double, 16)
            SAIL_CASE(double, 24) SAIL_CASE(double, 32)
        }
    }
#undef SAIL_CASE
}

sail_status launch_sweep(sail_problem *p, int k0, int k1, const SweepParams &sp, hipStream_t stream)
{
    const int mode = sp.walk_len > 0 ? kSweepWalk : sweep_traced(p, k0, k1) ? kSweepTraced : kSweepFast;
    const SweepPlan s = plan_alone(p, mode, sp.walk_len);
    const SweepArgs a = make_sweep_args(p, k0, k1, sp, s);
    const int blocks = sweep_blocks(p, s);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (p->timing) {
        if (p->ev_used == p->ev_start.size()) {
            hipEvent_t x, y;
            SAIL_HIP(hipEventCreate(&x));
            SAIL_HIP(hipEventCreate(&y));
            p->ev_start.push_back(x);
            p->ev_stop.push_back(y);
        }
        e0 = p->ev_start[p->ev_used];
        e1 = p->ev_stop[p->ev_used];
        p->ev_used++;
        SAIL_HIP(hipEventRecord(e0, stream));
    }
    with_basis_class(p->precision, p->dims(p->precision), [&](auto r, auto m) {
        launch_sweep_m<decltype(r), decltype(m)::value>(a, blocks, s, mode, stream);
    });
    SAIL_HIP(hipGetLastError());
    if (p->timing) SAIL_HIP(hipEventRecord(e1, stream));
    return SAIL_OK;
}

// The basis of the weighted columns and everything built from the kernel: the
// exact columns E, the columns in the basis, and the sweep's residue tables.
//
// Basis: a greedy (pivoted, twice orthogonalised Gram-Schmidt) selection of
// columns sqrt(wh_i) e^{-omega_j tau_i}, each taken relative to its own norm,
// then rotated to the principal directions of the selection's sample (one-sided
// Jacobi), of which the first are kept, as many as leave less than kBasisTol64
// of any column, filled up to the whole chunks they are stored in.  The sweep drops
// the product of two such residuals, so the scalar products of the FP64 loop
// are good to kBasisTol64^2 = 1e-14 of the norms at worst.  That must not exceed
// what summing over columns from a recurrence along tau in doubles left (in units of
// the condition scale, spectra of two bins, which resolve the columns best, 600
// grids of 32 to 900 bins and 16 to 256 times): 16 dimensions and more leave 2e-17 to
// 9e-17 rms and at most 2.0e-15, the recurrence 8e-17 to 6e-16 and 5e-16 to 6e-15, the
// larger its grids; at most 0.56 times the recurrence's maximum on any grid.  The
// small grids that 8 dimensions hold to 1e-7 had a recurrence as short as
// they (1.0e-15 to 2.1e-15) against up to 7e-15 left out, so these must hold to
// kBasisTolLeast (else 16: 1.2e-16).  The FP32 loop takes
// the first vectors, up to kBasisTol32 (squared 1e-8, below its rounding).  The
// selection runs on the host on kBasisSample columns spread over the grid; the
// device projects every column on it, and those found outside their span join
// the sample.
constexpr double kBasisTol64 = 1e-7, kBasisTolLeast = 2e-8, kBasisTol32 = 1e-4, kBasisGreedy = 1e-8;
constexpr int kBasisSample = 64;
// Dimensions at most.  Decaying kernels give 5 to 25.  Weights that turn the columns
// into separate Gaussians give most.  Equally wide ones are some sqrt(32 W) / pi, W the
// range of omega tau, which is below 1450 where the columns' norms fit a double: 73 (in
// FP32 56) computed there; ones that widen with tau are more: 107 (78) the most that a
// search over such weights found.
constexpr int kBasisMost = 4 * kDims64[6], kBasisMost32 = 4 * kDims32[5];
constexpr int kBasisReckoned = 96;  // in footprints

double dot(const double *x, const double *y, int n)
{
    double s[8] = {};
    int i = 0;
    for (; i + 8 <= n; i += 8)
        for (int t = 0; t < 8; ++t) s[t] += x[i + t] * y[i + t];
    for (; i < n; ++i) s[0] += x[i] * y[i];
    return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
}

// Rotates the rows of b (n rows of m) to mutually orthogonal ones, largest
// first, by one-sided Jacobi; r (n x n) receives the rotation.
void principal_rows(std::vector<std::vector<double>> &b, std::vector<std::vector<double>> &r)
{
    const int n = (int)b.size(), m = n ? (int)b[0].size() : 0;
    r.assign(n, std::vector<double>(n, 0.0));
    for (int i = 0; i < n; ++i) r[i][i] = 1.0;
    for (int sweep = 0; sweep < 12; ++sweep) {
        bool moved = false;
        for (int i = 0; i < n; ++i)
            for (int j = i + 1; j < n; ++j) {
                const double a = dot(b[i].data(), b[i].data(), m), d = dot(b[j].data(), b[j].data(), m);
                const double g = dot(b[i].data(), b[j].data(), m);
                if (!(std::fabs(g) > 1e-10 * std::sqrt(a * d)) || !(a * d > 0.0)) continue;
                moved = true;
                const double z = (d - a) / (2.0 * g);
                const double t = (z >= 0.0 ? 1.0 : -1.0) / (std::fabs(z) + std::sqrt(1.0 + z * z));
                const double cs = 1.0 / std::sqrt(1.0 + t * t), sn = cs * t;
                auto turn = [&](std::vector<double> &x, std::vector<double> &y) {
                    for (size_t k = 0; k < x.size(); ++k) {
                        const double u = x[k], v = y[k];
                        x[k] = cs * u - sn * v;
                        y[k] = sn * u + cs * v;
                    }
                };
                turn(b[i], b[j]);
                turn(r[i], r[j]);
            }
        if (!moved) break;
    }
    std::vector<int> by(n);
    std::vector<double> size(n);
    for (int i = 0; i < n; ++i) {
        by[i] = i;
        size[i] = dot(b[i].data(), b[i].data(), m);
    }
    std::stable_sort(by.begin(), by.end(), [&](int x, int y) { return size[x] > size[y]; });
    std::vector<std::vector<double>> br(n), rr(n);
    for (int i = 0; i < n; ++i) {
        br[i] = std::move(b[by[i]]);
        rr[i] = std::move(r[by[i]]);
    }
    b = std::move(br);
    r = std::move(rr);
}

class BasisSample {
public:
    BasisSample(const sail_problem *p, const std::vector<double> &sw) : p_(p), sw_(sw) {}

    // takes column j into the sample; false if it was there or spans nothing
    bool take(int j)
    {
        if (std::find(bins_.begin(), bins_.end(), j) != bins_.end()) return false;
        const int n = p_->n_tau;
        std::vector<double> v(n);
        for (int i = 0; i < n; ++i) v[i] = sw_[i] * std::exp(-p_->omega[j] * p_->tau[i]);
        const double norm = std::sqrt(dot(v.data(), v.data(), n));
        if (!(norm > 0.0) || !std::isfinite(norm)) return false;
        for (auto &x : v) x /= norm;
        column_.push_back(v);
        for (const auto &u : q_) {
            const double s = dot(u.data(), v.data(), n);
            for (int i = 0; i < n; ++i) v[i] -= s * u[i];
        }
        rest_.push_back(std::move(v));
        bins_.push_back(j);
        return true;
    }

    // extends the selection until it spans the sample to kBasisGreedy, and
    // returns it rotated: [vectors][n_tau], orthonormal; more vectors than columns of
    // the first sample only if `turn`
    std::vector<std::vector<double>> vectors(bool turn)
    {
        const int n = p_->n_tau, most = std::min(p_->n_omega, n);
        while ((int)q_.size() < most) {
            int pick = -1;
            double big = kBasisGreedy;
            for (size_t i = 0; i < rest_.size(); ++i) {
                const double v = std::sqrt(dot(rest_[i].data(), rest_[i].data(), n));
                if (v > big) {
                    big = v;
                    pick = (int)i;
                }
            }
            if (pick < 0) break;
            std::vector<double> u = rest_[pick];
            for (int pass = 0; pass < 2; ++pass)
                for (const auto &w : q_) {
                    const double s = dot(w.data(), u.data(), n);
                    for (int i = 0; i < n; ++i) u[i] -= s * w[i];
                }
            const double un = std::sqrt(dot(u.data(), u.data(), n));
            if (!(un > 0.5 * big)) {  // nothing but rounding was left
                std::fill(rest_[pick].begin(), rest_[pick].end(), 0.0);
                continue;
            }
            for (auto &x : u) x /= un;
            for (auto &v : rest_) {
                const double s = dot(u.data(), v.data(), n);
                for (int i = 0; i < n; ++i) v[i] -= s * u[i];
            }
            q_.push_back(std::move(u));
        }
        std::vector<std::vector<double>> q = q_;
        const int dims = (int)q.size();
        // principal directions of the sampled columns
        if (dims <= kBasisSample || turn) {
            std::vector<std::vector<double>> rows(dims), r;
            for (int d = 0; d < dims; ++d)
                for (const auto &v : column_) rows[d].push_back(dot(q_[d].data(), v.data(), n));
            principal_rows(rows, r);
            for (int d = 0; d < dims; ++d) {
                std::fill(q[d].begin(), q[d].end(), 0.0);
                for (int e = 0; e < dims; ++e)
                    for (int i = 0; i < n; ++i) q[d][i] += r[d][e] * q_[e][i];
            }
        }
        // the rotations leave q orthonormal to some 1e-15 only, which S2 would
        // show: once more, in 80 bits
        for (int d = 0; d < dims; ++d) {
            std::vector<long double> u(q[d].begin(), q[d].end());
            for (int e = 0; e < d; ++e) {
                long double t = 0.0L;
                for (int i = 0; i < n; ++i) t += q[e][i] * u[i];
                for (int i = 0; i < n; ++i) u[i] -= t * q[e][i];
            }
            long double t = 0.0L;
            for (int i = 0; i < n; ++i) t += u[i] * u[i];
            t = std::sqrt(t);
            for (int i = 0; i < n; ++i) q[d][i] = (double)(u[i] / t);
        }
        return q;
    }

private:
    const sail_problem *p_;
    const std::vector<double> &sw_;
    std::vector<int> bins_;                             // the sampled columns
    std::vector<std::vector<double>> column_, rest_, q_;  // they, relative to their norms; what q_ leaves of them
};

sail_status build_tables(sail_problem *p)
{
    const int No = p->n_omega, Nt = p->n_tau;
    const size_t pairs = 2 * (size_t)No - 1;
    // one array: what the host makes (omega, tau, wh, Phit, cn, cfac), then the
    // pass's vectors and results, then the tables of bins and pair sums
    auto whole = [](size_t n) { return (n + 31) & ~(size_t)31; };
    const size_t o_tau = whole(No), o_wh = o_tau + whole(Nt), o_Phit = o_wh + whole(Nt), o_cn = o_Phit + whole(Nt),
                 o_cfac = o_cn + whole(Nt), o_proj = o_cfac + whole(Nt), o_worst = o_proj + (size_t)kBasisPass * Nt, o_tail = o_worst + kBasisPass,
                 o_bin = o_tail + whole(No), o_GH = o_bin + 4 * whole(No), size = o_GH + 2 * pairs;
    sail_status st;
    if ((st = dalloc(&p->d_tab, size))) return st;
    double *tab = p->d_tab;
    p->d_omega = tab;
    p->d_wh = tab + o_wh;
    p->d_Phit = tab + o_Phit;
    p->d_cfac = tab + o_cfac;
    p->d_bin = tab + o_bin;
    p->d_GH = tab + o_GH;
    std::vector<double> h(o_proj, 0.0), sw(Nt);
    std::copy(p->omega.begin(), p->omega.end(), h.begin());
    std::copy(p->tau.begin(), p->tau.end(), h.begin() + o_tau);
    double C = 0.0;
    for (int i = 0; i < Nt; ++i) {
        const double wh = p->w[i] * p->cfac[i] * p->cfac[i], Phit = p->F[i] / p->cfac[i];
        h[o_wh + i] = wh;
        h[o_Phit + i] = Phit;
        h[o_cn + i] = -(2.0 * wh) * Phit;
        h[o_cfac + i] = p->cfac[i];
        sw[i] = std::sqrt(wh);
        C += wh * Phit * Phit;
    }
    p->tC = C;
    p->tw0 = p->omega[0];
    p->tdW = (p->omega[No - 1] - p->omega[0]) / (double)(No - 1);
    SAIL_HIP(hipMemcpy(tab, h.data(), sizeof(double) * h.size(), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_pair_sums, dim3((unsigned)pairs), dim3(64), 0, nullptr, Nt, 2.0 * p->tw0, p->tdW,
                       (const double *)(tab + o_tau), (const double *)p->d_wh, (double2 *)p->d_GH);
    SAIL_HIP(hipGetLastError());
    TableArgs a{};
    a.n_omega = No;
    a.n_tau = Nt;
    a.omega = tab;
    a.tau = tab + o_tau;
    a.wh = p->d_wh;
    a.cn = tab + o_cn;
    a.proj = tab + o_proj;
    a.worst = tab + o_worst;
    a.tail = tab + o_tail;
    a.bin = (double4 *)p->d_bin;
    std::vector<std::vector<double>> q;
    std::vector<double> up((size_t)kBasisPass * Nt);
    int loaded = -1;  // first vector of the pass on the device
    auto pass = [&](int d0, int nd) -> sail_status {
        a.d0 = d0;
        a.nd = nd;
        if (loaded != d0) {
            for (int d = 0; d < nd; ++d)
                for (int i = 0; i < Nt; ++i) up[(size_t)d * Nt + i] = sw[i] * q[d0 + d][i];
            SAIL_HIP(hipMemcpy(tab + o_proj, up.data(), sizeof(double) * (size_t)nd * Nt, hipMemcpyHostToDevice));
            loaded = d0;
        }
        hipLaunchKernelGGL(k_tables, dim3(No), dim3(kThreads), sizeof(double) * Nt, nullptr, a);
        SAIL_HIP(hipGetLastError());
        return SAIL_OK;
    };
    BasisSample sample(p, sw);
    const int ns = std::min(No, kBasisSample);
    for (int i = 0; i < ns; ++i) sample.take((int)((int64_t)i * (No - 1) / std::max(1, ns - 1)));
    std::vector<double> got(kBasisPass + No), worst;
    int dims64, dims32;
    for (bool turn = false;;) {
        q = sample.vectors(turn);
        loaded = -1;
        // what every column holds from each vector on, last vectors first
        const int dims = (int)q.size();
        worst.assign(dims, 0.0);
        std::fill(got.begin(), got.end(), 0.0);
        SAIL_HIP(hipMemcpy(tab + o_worst, got.data(), sizeof(double) * got.size(), hipMemcpyHostToDevice));
        for (int d0 = (dims - 1) / kBasisPass * kBasisPass; dims > 0 && d0 >= 0; d0 -= kBasisPass) {
            const int nd = std::min(kBasisPass, dims - d0);
            if ((st = pass(d0, nd))) return st;
            SAIL_HIP(hipMemcpy(got.data(), tab + o_worst, sizeof(double) * got.size(), hipMemcpyDeviceToHost));
            std::copy(got.begin(), got.begin() + nd, worst.begin() + d0);
        }
        // columns outside the span: take some and select on
        std::vector<int> out;
        for (int j = 0; dims > 0 && j < No; ++j)
            if (1.0 - got[kBasisPass + j] > 0.25 * kBasisTol64 * kBasisTol64) out.push_back(j);
        bool more = false;
        const int want = std::min<int>((int)out.size(), 16);
        for (int i = 0; i < want; ++i) more |= sample.take(out[(size_t)i * out.size() / want]);
        if (more) continue;
        dims64 = dims32 = dims;
        for (int d = dims - 1; d >= 1; --d) {
            const double tol = d <= 4 * kDims64[0] ? kBasisTolLeast : kBasisTol64;
            if (worst[d] <= tol * tol) dims64 = d;
            if (worst[d] <= kBasisTol32 * kBasisTol32) dims32 = d;
        }
        // (500 bins, 512 times under weights whose columns widen along tau: 106 and 99
        // as selected, 98 and 72 rotated)
        if ((dims64 <= kBasisMost && dims32 <= kBasisMost32) || turn) break;
        turn = true;
    }
    const int dims = (int)q.size();
    if (dims64 > kBasisMost || dims32 > kBasisMost32)
        return fail(SAIL_ENUMERIC, "the weighted columns span too many dimensions");
    p->dims64 = round_dims(SAIL_FP64, dims64);
    p->dims32 = round_dims(SAIL_FP32, dims32);
    const int ec = p->echunk = chunk_stride<double>(p->dims64), kept = std::min(dims, 4 * p->dims64);
    uint64_t id = 0xcbf29ce484222325ull;  // FNV-1a, word by word
    for (int d = 0; d < kept; ++d)
        for (int i = 0; i < Nt; ++i) {
            const double v = sw[i] * q[d][i];
            uint64_t x;
            std::memcpy(&x, &v, sizeof x);
            id = (id ^ x) * 0x100000001b3ull;
        }
    p->basis_id = id;
    if ((st = dalloc(&p->d_E, (size_t)No * p->cols()))) return st;
    a.E = p->d_E;
    a.cols = p->cols();
    a.echunk = ec;
    int d0 = 0;
    do {
        if ((st = pass(d0, std::min(kBasisPass, kept - d0)))) return st;
        d0 += kBasisPass;
    } while (d0 < kept);
    return SAIL_OK;
}

constexpr int kDefaultTile = 16;

// The nominal lane layout: TPL tau points per lane (16 unless requested
// otherwise; more only when N_tau needs it), a power-of-two number of lanes per
// walker, tau padded to lanes * TPL; and the columns in the loop precision.
sail_status build_layout(sail_problem *p, int precision)
{
    const int n_tau = p->n_tau;
    const int tpl_max = precision == SAIL_FP32 ? 32 : 16;
    int tpl = kDefaultTile;
    auto tile_ok = [&](int v) { return v == tpl_max || v == tpl_max / 2 || v == tpl_max / 4; };
    if (tile_ok(p->tpl_hint)) {
        tpl = p->tpl_hint;
    } else if (const char *env = std::getenv("SAIL_TPL")) {
        const int v = std::atoi(env);
        if (tile_ok(v)) tpl = v;
    }
    int lanes = next_pow2((n_tau + tpl - 1) / tpl);
    while (lanes > 64 && tpl < tpl_max) {
        tpl *= 2;
        lanes = next_pow2((n_tau + tpl - 1) / tpl);
    }
    if (lanes > 64) return fail(SAIL_EINVAL, "n_tau too large for the sweep layout");
    p->tpl = tpl;
    p->lanes = lanes;
    p->ntau_pad = lanes * tpl;
    return SAIL_OK;
}

// The sweep's columns in the loop precision.
sail_status build_columns(sail_problem *p, int precision, hipStream_t stream)
{
    const int n_omega = p->n_omega, n_tau = p->n_tau;
    if (p->layout_precision == precision) return SAIL_OK;
    dfree(p->d_col);
    p->layout_precision = -1;
    const int ec = p->echunk, ck = p->chunk(precision);
    const size_t n = (size_t)n_omega * 4 * ck, rsz = precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    char *col = nullptr;
    const sail_status st = dalloc(&col, rsz * n);
    if (st) return st;
    p->d_col = col;
    auto columns = [&](auto *to) {
        hipLaunchKernelGGL(k_columns, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, (int)n, n_tau,
                           p->cols(), ec, ck, (const double *)p->d_E, to);
    };
    if (precision == SAIL_FP32) columns((float *)col);
    else columns((double *)col);
    SAIL_HIP(hipGetLastError());
    p->layout_precision = precision;
    return SAIL_OK;
}

sail_status check_schedule_params(const sail_schedule *sc, int first_sweep, int n_sweeps)
{
    if (!sc) return fail(SAIL_EINVAL, "NULL schedule");
    if (!sc->T || sc->n_T <= 0) return fail(SAIL_EINVAL, "empty temperature schedule");
    if (first_sweep < 0 || n_sweeps < 0 || first_sweep + n_sweeps > sc->n_T) return fail(SAIL_EINVAL, "sweeps outside the schedule");
    if (sc->branch_every <= 0 || sc->resync_every <= 0 || sc->branch_every % sc->resync_every != 0)
        return fail(SAIL_EINVAL, "resync_every must divide branch_every");
    if (!(sc->eps0 > 0.0 && sc->eps0 < 1.0)) return fail(SAIL_EINVAL, "eps0 must lie in (0, 1)");
    if (!(sc->amp_avg > 0.0 && sc->amp_avg <= 1.0)) return fail(SAIL_EINVAL, "amp_avg must lie in (0, 1]");
    if (!(sc->amp_p > 0.0) || sc->amp_m < 0) return fail(SAIL_EINVAL, "bad amplitude parameters");
    if (!(sc->branch_fraction >= 0.0 && sc->branch_fraction < 1.0)) return fail(SAIL_EINVAL, "bad branch fraction");
    if (!(sc->imprint_t >= 0.0 && sc->imprint_t <= 1.0)) return fail(SAIL_EINVAL, "imprint_t must lie in [0, 1]");
    if (sc->walk_len < 0 || sc->walk_len > kMaxWalk) return fail(SAIL_EINVAL, "walk_len must lie in [0, 64]");
    if (sc->t_units != 0 && sc->t_units != 1) return fail(SAIL_EINVAL, "bad t_units");
    if (!(sc->smooth >= 0.0 && sc->smooth <= 0.5)) return fail(SAIL_EINVAL, "smooth must lie in [0, 0.5]");
    if (sc->adaptive != 0 && sc->adaptive != 1) return fail(SAIL_EINVAL, "adaptive must be 0 or 1");
    if ((sc->self_cool != 0 && sc->self_cool != 1) || sc->boil_blocks < 0 || sc->cool_blocks < 1)
        return fail(SAIL_EINVAL, "self-cooling needs self_cool 0 or 1, boil_blocks >= 0, cool_blocks >= 1");
    for (int k = first_sweep; k < first_sweep + n_sweeps; ++k)
        if (!(sc->T[k] > 0.0) || !std::isfinite(sc->T[k])) return fail(SAIL_EINVAL, "temperatures must be positive and finite");
    return SAIL_OK;
}

sail_status check_schedule(const sail_problem *p, const sail_schedule *sc, int first_sweep, int n_sweeps)
{
    if (!p || !sc) return fail(SAIL_EINVAL, "NULL argument");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    if (p->n_walkers > kBranchMaxWalkers) return fail(SAIL_EINVAL, "too many walkers for the branching kernel");
    return check_schedule_params(sc, first_sweep, n_sweeps);
}

// Event log capacity for sweeps up to `last` and the absolute temperatures
// of the schedule on the device (synchronises `stream`).
sail_status prepare_schedule(sail_problem *p, const sail_schedule *sc, int last, hipStream_t stream)
{
    sail_status st;
    if ((st = ensure_events(p, last / sc->branch_every + 1, stream))) return st;
    if (sc->self_cool) {
        // the temperatures are computed on the device block by block
        if (sc->n_T > p->cap_T) {
            SAIL_HIP(hipStreamSynchronize(stream));
            dfree(p->d_Tabs);
            p->self_T_end = 0;
            if ((st = dalloc(&p->d_Tabs, sc->n_T))) {
                p->cap_T = 0;
                return st;
            }
            p->cap_T = sc->n_T;
        }
        p->h_Tabs.clear();
        return SAIL_OK;
    }
    std::vector<double> Tabs(sc->T, sc->T + sc->n_T);
    if (sc->t_units == 0)
        for (auto &v : Tabs) v = v * p->chi2_unit;
    if (Tabs == p->h_Tabs) return SAIL_OK;  // already on the device
    SAIL_HIP(hipStreamSynchronize(stream));  // sweeps in flight may read d_Tabs
    p->h_Tabs.clear();
    if (sc->n_T > p->cap_T) {
        dfree(p->d_Tabs);
        if ((st = dalloc(&p->d_Tabs, sc->n_T))) {
            p->cap_T = 0;
            return st;
        }
        p->cap_T = sc->n_T;
    }
    SAIL_HIP(hipMemcpy(p->d_Tabs, Tabs.data(), sizeof(double) * sc->n_T, hipMemcpyHostToDevice));
    p->h_Tabs = std::move(Tabs);
    p->self_T_end = 0;
    return SAIL_OK;
}

// The largest padded time grid any candidate layout of this precision takes.
size_t max_padding(int n_tau, int precision)
{
    const int tmin = precision == SAIL_FP32 ? 16 : 8;
    size_t ntp = 0;
    for (int t = tmin; t <= 2 * tmin; t *= 2) ntp = std::max(ntp, (size_t)next_pow2((n_tau + t - 1) / t) * t);
    return ntp;
}

// Device bytes of a problem's tables, each rounded as the allocator rounds it;
// the basis of min(n_tau, n_omega, kBasisReckoned) dimensions at most.
size_t table_bytes(int n_omega, int n_tau, int precision)
{
    const size_t rsz = precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t No = (size_t)n_omega;
    const int most = std::min(std::min(n_tau, n_omega), kBasisReckoned);
    const size_t d64 = 4 * (size_t)chunk_stride<double>(round_dims(SAIL_FP64, most));
    const size_t d32 = 4 * (size_t)chunk_stride<float>(round_dims(SAIL_FP32, most));
    return sizeof(double) * (6 * No + No * (n_tau + d64) + (5 + kBasisPass) * (size_t)n_tau + kBasisPass + 2 * (2 * No - 1)) +
           rsz * No * (precision == SAIL_FP32 ? d32 : d64) +
           12 * 256;
}

// Layouts chosen by the autotuner, per (device architecture, n_omega, n_tau,
// n_walkers, precision, device to itself or shared).  With SAIL_TUNE_CACHE
// naming a file, the choices persist across processes: the file is read at
// the first lookup, and every new choice is appended as one line
// "<tag> <arch> <n_omega> <n_tau> <n_walkers> <precision> <tau per lane>",
// tag sail-tune-v1 for a shared device, sail-tune-alone-v1 for a device to
// itself (malformed lines are ignored).
using TuneKey = std::tuple<std::string, int, int, int, int, bool>;
constexpr const char *kTuneTag[2] = {"sail-tune-v1", "sail-tune-alone-v1"};
std::mutex g_tune_mu;
std::map<TuneKey, int> g_tuned;
bool g_tune_loaded = false;

std::string device_arch(int device)
{
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return "unknown";
    std::string a = prop.gcnArchName;
    const size_t colon = a.find(':');
    return colon == std::string::npos ? a : a.substr(0, colon);
}

void load_tune_cache()  // under g_tune_mu
{
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char *path = std::getenv("SAIL_TUNE_CACHE");
    if (!path || !*path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;
    char tag[32], arch[64];
    int no, nt, nw, pr, tpl;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        if (std::sscanf(line, "%31s %63s %d %d %d %d %d", tag, arch, &no, &nt, &nw, &pr, &tpl) != 7) continue;
        const std::string t(tag);
        if ((t != kTuneTag[0] && t != kTuneTag[1]) || tpl <= 0) continue;
        g_tuned[TuneKey(arch, no, nt, nw, pr, t == kTuneTag[1])] = tpl;
    }
    std::fclose(f);
}

bool tuned_layout(int device, int n_omega, int n_tau, int n_walkers, int precision, int *tpl, bool alone = false)
{
    const std::string arch = device_arch(device);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_tune_cache();
    auto it = g_tuned.find(TuneKey(arch, n_omega, n_tau, n_walkers, precision, alone));
    if (it == g_tuned.end()) return false;
    *tpl = it->second;
    return true;
}

void remember_layout(int device, int n_omega, int n_tau, int n_walkers, int precision, int tpl, bool alone)
{
    const std::string arch = device_arch(device);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_tune_cache();
    g_tuned[TuneKey(arch, n_omega, n_tau, n_walkers, precision, alone)] = tpl;
    const char *path = std::getenv("SAIL_TUNE_CACHE");
    if (!path || !*path) return;
    if (FILE *f = std::fopen(path, "a")) {
        std::fprintf(f, "%s %s %d %d %d %d %d\n", kTuneTag[alone], arch.c_str(), n_omega, n_tau, n_walkers, precision,
                     tpl);
        std::fclose(f);
    }
}

// The sweeps from k run in one launch up to the next resync boundary.
int segment_end(const sail_schedule *sc, int k, int last)
{
    const int kend = (k / sc->resync_every + 1) * sc->resync_every;
    return kend > last ? last : kend;
}

// --------------------------------------------------------------------------
// Many problems advanced together.  A round takes every unfinished job to
// its next resync boundary: one sweep launch per (precision, basis class, mode)
// holds the workgroups of all of them, then one launch each for the
// renormalising resync, the branching solves and the imprint + target resync
// of the jobs that reached such a boundary.  Every job runs exactly the
// kernels' per-problem code on its own state, so its result is bit-identical
// to running it alone.  Per-round descriptors are packed into one pinned
// staging slot and copied with a single H2D copy; a ring of slots lets the
// host run a few rounds ahead of the device.
// --------------------------------------------------------------------------
struct BatchJob {
    sail_problem *p = nullptr;
    sail_schedule sc{};
    int k = 0, last = 0;
};

constexpr int kSweepGroups = 2 * 6 * 3;  // precisions x basis classes of each x modes

struct StageRing {
    static constexpr int kSlots = 4;
    char *h[kSlots] = {};
    char *d[kSlots] = {};
    hipEvent_t done[kSlots] = {};
    size_t cap = 0;
    int next = 0;

    // A round puts, per job, one sweep descriptor, up to three resync
    // descriptors (renormalise; imprint after a branching event; smoothing)
    // and one branching descriptor, plus one workgroup offset per launch
    // list the job joins (one sweep list, three resync passes).  Each put
    // starts on a 64-byte boundary and each launch list ends with one extra
    // offset: at most kMaxPuts puts per round (kSweepGroups sweep groups x 2, 2
    // precisions x 3 resync passes x kResyncClasses LDS classes x 2, one
    // branching array, one block-log array).
    static constexpr size_t kMaxPuts = kSweepGroups * 2 + 2 * 3 * kResyncClasses * 2 + 1 + 1;
    static size_t bytes_per_job()
    {
        return sizeof(SweepArgs) + 3 * sizeof(ResyncArgs) + sizeof(BranchArgs) + sizeof(BlockLogArgs) + 4 * sizeof(int);
    }
    static size_t bytes_for(int n_jobs) { return (size_t)n_jobs * bytes_per_job() + kMaxPuts * (64 + sizeof(int)); }
    sail_status reserve(int n_jobs)
    {
        const size_t need = bytes_for(n_jobs);
        if (need <= cap) return SAIL_OK;
        release();
        for (int i = 0; i < kSlots; ++i) {
            if (hipHostMalloc((void **)&h[i], need, hipHostMallocDefault) != hipSuccess) {
                h[i] = nullptr;
                release();
                return fail(SAIL_ENOMEM, "pinned staging buffer");
            }
            if (raw_alloc((void **)&d[i], need) != hipSuccess) {
                d[i] = nullptr;
                release();
                return fail(SAIL_ENOMEM, "device staging buffer");
            }
            if (hipEventCreateWithFlags(&done[i], hipEventDisableTiming) != hipSuccess) {
                done[i] = nullptr;
                release();
                return fail(SAIL_EDEVICE, "staging event");
            }
        }
        cap = need;
        return SAIL_OK;
    }
    void release()
    {
        for (int i = 0; i < kSlots; ++i) {
            if (done[i]) (void)hipEventSynchronize(done[i]);
            if (h[i]) (void)hipHostFree(h[i]);
            if (d[i]) raw_free(d[i]);
            if (done[i]) (void)hipEventDestroy(done[i]);
            h[i] = d[i] = nullptr;
            done[i] = nullptr;
        }
        cap = 0;
    }
};

// Sequential writer into a staging slot; device addresses mirror host ones.
// A put that would pass the slot's end copies nothing and marks the round as
// overflowed (the caller then fails the round before anything is launched).
struct Stager {
    char *h, *d;
    size_t off = 0, cap;
    bool overflow = false;
    template <typename T>
    T *put(const T *src, size_t n)
    {
        const size_t at = (off + 63) & ~(size_t)63;
        if (at + sizeof(T) * n > cap) {
            overflow = true;
            return nullptr;
        }
        T *dst = (T *)(d + at);
        std::memcpy(h + at, src, sizeof(T) * n);
        off = at + sizeof(T) * n;
        return dst;
    }
};

// HIP events around the shared sweep launches; completed pairs are folded
// into the running total without waiting on launches still in flight.
struct SweepTimer {
    int enabled = 0;
    std::deque<std::pair<hipEvent_t, hipEvent_t>> pending;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
    double ms = 0.0;
    int64_t n = 0;
    sail_status begin(hipStream_t stream, hipEvent_t *e1)
    {
        *e1 = nullptr;
        if (!enabled) return SAIL_OK;
        std::pair<hipEvent_t, hipEvent_t> ev;
        if (pool.empty()) {
            SAIL_HIP(hipEventCreate(&ev.first));
            SAIL_HIP(hipEventCreate(&ev.second));
        } else {
            ev = pool.back();
            pool.pop_back();
        }
        SAIL_HIP(hipEventRecord(ev.first, stream));
        pending.push_back(ev);
        *e1 = ev.second;
        return SAIL_OK;
    }
    sail_status harvest(bool block)
    {
        while (!pending.empty()) {
            const auto ev = pending.front();
            const hipError_t q = block ? hipEventSynchronize(ev.second) : hipEventQuery(ev.second);
            if (q == hipErrorNotReady) break;
            if (q != hipSuccess) return fail(SAIL_EDEVICE, std::string("sweep timing: ") + hipGetErrorString(q));
            float x = 0.f;
            SAIL_HIP(hipEventElapsedTime(&x, ev.first, ev.second));
            ms += x;
            n++;
            pending.pop_front();
            pool.push_back(ev);
        }
        return SAIL_OK;
    }
    sail_status total(double *out_ms, int64_t *out_n, bool reset)
    {
        sail_status st = harvest(true);
        if (st) return st;
        if (out_ms) *out_ms = ms;
        if (out_n) *out_n = n;
        if (reset) {
            ms = 0.0;
            n = 0;
        }
        return SAIL_OK;
    }
    ~SweepTimer()
    {
        for (auto &e : pending) pool.push_back(e);
        for (auto &e : pool) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
    }
};

struct Launch {
    int kind, blocks, n;
    const void *args;
    const int *first;
    size_t shm;
    int cls = 0, mode = 0, threads = kThreads;  // sweeps only
    int wpb = 8;  // resyncs only
    int lanes = 4, near = 0;  // sweeps only
};

template <typename R, int M>
void launch_sweep_batched_m(const Launch &L, const SweepArgs *jobs, hipStream_t stream)
{
    const dim3 grid(L.blocks), thr(L.threads);
    constexpr bool WIDE = wide_basis(M);
    if (L.mode == kSweepFast) {
        hipLaunchKernelGGL((k_sweep_split_batched<R, M>), grid, thr, L.shm, stream, jobs, L.first, L.n, L.near);
    } else if (L.mode == kSweepTraced) {
        hipLaunchKernelGGL((k_sweep_batched<R, M, kSweepTraced, WIDE ? 16 : 4>), grid, thr, L.shm, stream, jobs, L.first, L.n);
    } else if constexpr (WIDE) {
        hipLaunchKernelGGL((k_sweep_batched<R, M, kSweepWalk, 16>), grid, thr, L.shm, stream, jobs, L.first, L.n);
    } else if (L.lanes == 4) {
        hipLaunchKernelGGL((k_sweep_batched<R, M, kSweepWalk, 4>), grid, thr, L.shm, stream, jobs, L.first, L.n);
    } else {
        hipLaunchKernelGGL((k_sweep_batched<R, M, kSweepWalk, 8>), grid, thr, L.shm, stream, jobs, L.first, L.n);
    }
}

void launch_sweep_batched(const Launch &L, const SweepArgs *jobs, hipStream_t stream)
{
    with_basis_class(L.kind, L.cls, [&](auto r, auto m) {
        launch_sweep_batched_m<decltype(r), decltype(m)::value>(L, jobs, stream);
    });
}

// Enqueues one round for the unfinished jobs in `jobs` (advancing their k).
sail_status batch_round(std::vector<BatchJob *> &jobs, StageRing &ring, SweepTimer &timer, hipStream_t stream)
{
    std::vector<BatchJob *> act;
    for (auto *j : jobs)
        if (j->k < j->last) act.push_back(j);
    if (act.empty()) return SAIL_OK;
    sail_status st;
    if ((st = ring.reserve((int)act.size()))) return st;
    const int slot = ring.next;
    ring.next = (ring.next + 1) % StageRing::kSlots;
    SAIL_HIP(hipEventSynchronize(ring.done[slot]));  // the copy that last read this slot has finished
    Stager sg{ring.h[slot], ring.d[slot], 0, ring.cap};

    std::vector<int> kend(act.size());
    for (size_t i = 0; i < act.size(); ++i) kend[i] = segment_end(&act[i]->sc, act[i]->k, act[i]->last);

    // sweep groups, heaviest workgroups first
    std::vector<Launch> sweeps, resyncs, targets, smooths;
    // A round ends with its longest jobs.  While SIMDs would be left without a
    // chain, those take 16 lanes a walker (1024 bins: 283 to 220 ns a proposal),
    // longest first, where their columns fit in LDS beside the larger records
    // (16 FP32 jobs of 9472 walkers, one round: 14.5 to 11.6 ms) and no compute unit
    // gets a second workgroup for it.
    std::vector<char> wide(act.size(), 0);
    // chain wavefronts of a problem at its fewest lanes a walker
    auto least_lanes = [](const sail_problem *p) { return wide_basis(p->dims(p->precision)) ? 16 : 4; };
    auto pairs_of = [&](const sail_problem *p) { return (p->n_walkers * least_lanes(p) + 63) / 64; };
    {
        int64_t simds = 4 * kCUs;
        std::vector<int> by(act.size());
        for (size_t i = 0; i < act.size(); ++i) {
            by[i] = (int)i;
            simds -= pairs_of(act[i]->p);
        }
        std::stable_sort(by.begin(), by.end(), [&](int x, int y) {
            return (int64_t)act[x]->p->n_omega * (kend[x] - act[x]->k) > (int64_t)act[y]->p->n_omega * (kend[y] - act[y]->k);
        });
        for (int i : by) {
            const int more = (act[i]->p->n_walkers + 3) / 4 - pairs_of(act[i]->p);
            if (more > simds) break;
            simds -= more;
            wide[i] = 1;
        }
    }
    // one sweep launch per (precision, basis class, mode); jobs of one
    // workload share theirs
    std::vector<int> group(act.size());
    for (size_t i = 0; i < act.size(); ++i) {
        const sail_problem *p = act[i]->p;
        const int mode = act[i]->sc.walk_len > 0 ? kSweepWalk : sweep_traced(p, act[i]->k, kend[i]) ? kSweepTraced : kSweepFast;
        group[i] = (p->precision * kBasisClasses + p->dims(p->precision)) * 3 + mode;
    }
    for (int g = 0; g < 2 * kBasisClasses * 3; ++g) {
        std::vector<int> idx;
        for (size_t i = 0; i < act.size(); ++i)
            if (group[i] == g) idx.push_back((int)i);
        if (idx.empty()) continue;
        std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) {
            const double cx = (double)act[x]->p->n_omega * (kend[x] - act[x]->k);
            const double cy = (double)act[y]->p->n_omega * (kend[y] - act[y]->k);
            return cx > cy;
        });
        Launch L{};
        L.mode = g % 3;
        L.cls = (g / 3) % kBasisClasses;
        L.kind = g / (3 * kBasisClasses);
        const bool walk = L.mode == kSweepWalk, split = L.mode == kSweepFast;
        L.threads = split ? 0 : kSweepThreads;
        L.lanes = least_lanes(act[idx[0]]->p);
        if (walk && L.lanes == 4) {
            // 8 lanes a walker, or 4 where 8 would leave a fifth of the last round
            // of wavefronts, two a SIMD, unused (256 bins, one step: 24 jobs of 1024
            // walkers 1.5 rounds, 1.54 against 1.71 ms; 1024 bins, 16 jobs of 4096
            // walkers 4 rounds, 8.4 against 7.2 ms)
            size_t waves = 0;
            for (int i : idx) waves += ((size_t)act[i]->p->n_walkers + 7) / 8;
            const size_t room = (size_t)2 * 4 * kCUs, rounds = (waves + room - 1) / room;
            L.lanes = rounds > 1 && waves * 5 < rounds * room * 4 ? 4 : 8;
        }
        std::vector<SweepArgs> sa;
        std::vector<int> first;
        std::vector<SweepPlan> plans;
        if (split) {
            // Pairs of wavefronts per workgroup: four share a compute unit's LDS copy
            // of the columns when workgroups abound; fewer while the workgroups do
            // not outnumber the compute units, each of which runs one (their
            // registers, and often their LDS, leave no room for a second): 24
            // FP64 jobs of 20736 walkers, with the columns of 1024 bins in LDS
            // beside two pairs, a round 27 ms, with four pairs for all 46 ms; 32
            // jobs of 512 bins, 300 walkers, two sweeps: 160 workgroups 377 us, 320
            // of two pairs 581 us.
            int pairs = 1;
            auto at = [&](int n) {
                size_t b = 0;
                for (int i : idx) b += ((size_t)pairs_of(act[i]->p) + n - 1) / n;
                return b;
            };
            while (pairs < 4 && at(pairs) > (size_t)kCUs) pairs *= 2;
            int total = 0;
            for (int i : idx) {
                const sail_problem *p = act[i]->p;
                // a job whose columns would not fit takes two pairs, hence fewer
                // records (1024 FP64 bins); not one of several, which leaves compute
                // units idle for long (1100 bins, four jobs of 4000 walkers: 2.28 ms, and
                // 1.41 ms with the columns in memory)
                SweepPlan s = plan_sweep(p, true, L.lanes, 128 * pairs, kLdsBytes, false, false, 0);
                for (int t = 64 * pairs; !s.columns_lds && t >= 256; t /= 2) {
                    const SweepPlan q = plan_sweep(p, true, L.lanes, t, kLdsBytes, false, false, 0);
                    if (q.columns_lds) s = q;
                }
                plans.push_back(s);
                total += sweep_blocks(p, s);
            }
            for (size_t n = 0; n < idx.size(); ++n) {
                const sail_problem *p = act[idx[n]]->p;
                for (int t = 4 * 128; wide[idx[n]] && L.lanes == 4 && t >= 128; t /= 2) {
                    const SweepPlan q = plan_sweep(p, true, 16, t, kLdsBytes, false, false, 0);
                    const int with = total - sweep_blocks(p, plans[n]) + sweep_blocks(p, q);
                    if (!q.columns_lds || with > kCUs) continue;
                    total = with;
                    plans[n] = q;
                    break;
                }
            }
        } else {
            for (int i : idx)
                plans.push_back(plan_sweep(act[i]->p, false, L.lanes, L.threads, kLdsBytes / 2, walk, false, act[i]->sc.walk_len));
        }
        int reading = 0;  // workgroups that read their columns from memory
        for (size_t n = 0; n < idx.size(); ++n) {
            const BatchJob *job = act[idx[n]];
            const sail_problem *p = job->p;
            const sail_schedule &sc = job->sc;
            const SweepPlan &s = plans[n];
            sa.push_back(make_sweep_args(p, job->k, kend[idx[n]],
                                         SweepParams{sc.eps0, sc.amp_p, sc.amp_avg, sc.amp_m, sc.walk_len}, s));
            first.push_back(L.blocks);
            L.blocks += sweep_blocks(p, s);
            if (!s.columns_lds) reading += sweep_blocks(p, s);
            L.shm = std::max(L.shm, s.shm);
            L.threads = std::max(L.threads, s.threads);
        }
        first.push_back(L.blocks);
        L.near = 2 * reading > L.blocks;
        L.n = (int)idx.size();
        L.args = sg.put(sa.data(), sa.size());
        L.first = sg.put(first.data(), first.size());
        sweeps.push_back(L);
    }
    // resyncs (renormalising) and imprint + target resyncs, by precision and
    // by the LDS their spectra need (one launch per class, so small problems
    // are not held to the LDS size, and occupancy, of the largest)
    std::vector<BranchArgs> ba;
    for (int prec = 0; prec < 2; ++prec) {
        // pass 0: renormalising resyncs; 1: imprint + target resyncs after the
        // branching solves; 2: smoothing of every walker (Sec. 2.6)
        for (int pass = 0; pass < 3; ++pass) for (int cls = 0; cls < kResyncClasses; ++cls) {
            std::vector<ResyncArgs> ra;
            std::vector<int> first;
            int blocks = 0, max_no = 0;
            size_t items = 0;
            for (const auto *j : act)
                if (j->p->precision == prec && resync_class(j->p->n_omega) == cls) {
                    items += (size_t)j->p->n_walkers;
                    max_no = std::max(max_no, j->p->n_omega);
                }
            const int wpb = resync_wpb(max_no, items);
            for (size_t i = 0; i < act.size(); ++i) {
                sail_problem *p = act[i]->p;
                const sail_schedule &sc = act[i]->sc;
                if (p->precision != prec) continue;
                if (resync_class(p->n_omega) != cls) continue;
                if (pass == 0 && kend[i] % sc.resync_every != 0) continue;
                if (pass >= 1 && kend[i] % sc.branch_every != 0) continue;
                if (pass == 2 && !(sc.smooth > 0.0)) continue;
                if (pass == 0) {
                    ra.push_back(make_resync_args(p, 1, nullptr, nullptr, p->n_walkers, nullptr, 0.0));
                    ra.back().drift = p->d_drift;  // the block log's drift, when it is on
                }
                else if (pass == 1)
                    ra.push_back(make_resync_args(p, 0, p->d_targets, p->d_npairs, p->n_walkers, p->d_donors,
                                                  sc.imprint_t, 0.0, sc.adaptive ? p->d_teff : nullptr));
                else
                    ra.push_back(make_resync_args(p, 1, nullptr, nullptr, p->n_walkers, nullptr, 0.0, sc.smooth));
                if (pass == 1)
                    ba.push_back(make_branch_args(p, sc.branch_fraction, kend[i] / sc.branch_every - 1, sc.adaptive,
                                                  sc.imprint_t));
                first.push_back(blocks);
                blocks += resync_blocks(p->n_walkers, wpb);
            }
            if (ra.empty()) continue;
            first.push_back(blocks);
            const ResyncArgs *dargs = sg.put(ra.data(), ra.size());
            const int *dfirst = sg.put(first.data(), first.size());
            (pass == 0 ? resyncs : pass == 1 ? targets : smooths)
                .push_back({prec, blocks, (int)ra.size(), dargs, dfirst, resync_shmem(max_no, wpb), 0, 0, kThreads, wpb});
        }
    }
    const BranchArgs *dbranch = ba.empty() ? nullptr : sg.put(ba.data(), ba.size());
    // block-log records of the jobs that keep one and end a resync interval
    std::vector<BlockLogArgs> bl;
    for (size_t i = 0; i < act.size(); ++i) {
        sail_problem *p = act[i]->p;
        const sail_schedule &sc = act[i]->sc;
        if (!p->d_blog || kend[i] % sc.resync_every != 0) continue;
        bl.push_back(BlockLogArgs{p->n_walkers, p->d_chi2, p->d_rate, p->d_drift, p->d_Tabs, kend[i],
                                  kend[i] % sc.branch_every == 0 ? kend[i] / sc.branch_every - 1 : -1,
                                  p->d_blog + (p->blog_total % p->blog_cap)});
    }
    const BlockLogArgs *dblog = bl.empty() ? nullptr : sg.put(bl.data(), bl.size());
    if (sg.overflow) return fail(SAIL_EDEVICE, "round descriptors exceed the staging slot");
    SAIL_HIP(hipMemcpyAsync(ring.d[slot], ring.h[slot], sg.off, hipMemcpyHostToDevice, stream));

    // self-cooling (Sec. 2.4): the temperature of each block that starts now
    for (auto *j : act) {
        const sail_schedule &sc = j->sc;
        if (!sc.self_cool || j->k % sc.branch_every != 0) continue;
        const int k1 = std::min(j->k + sc.branch_every, sc.n_T);
        hipLaunchKernelGGL(k_self_cool, dim3(1), dim3(kThreads), 0, stream, (const double *)j->p->d_chi2,
                           j->p->n_walkers, j->k / sc.branch_every, sc.boil_blocks, sc.cool_blocks, j->p->d_Tabs, j->k,
                           k1);
        SAIL_HIP(hipGetLastError());
        j->p->self_T_k0 = j->k;
        j->p->self_T_end = k1;
    }
    for (const Launch &L : sweeps) {
        hipEvent_t e1;
        if ((st = timer.begin(stream, &e1))) return st;
        launch_sweep_batched(L, (const SweepArgs *)L.args, stream);
        SAIL_HIP(hipGetLastError());
        if (e1) SAIL_HIP(hipEventRecord(e1, stream));
    }
    auto resync_launch = [&](const Launch &L) -> sail_status {
        const ResyncArgs *a = (const ResyncArgs *)L.args;
        if (L.kind == SAIL_FP32) launch_resync_k<float>(L.wpb, L.blocks, L.shm, stream, a, L.first, L.n);
        else launch_resync_k<double>(L.wpb, L.blocks, L.shm, stream, a, L.first, L.n);
        SAIL_HIP(hipGetLastError());
        return SAIL_OK;
    };
    for (const Launch &L : resyncs)
        if ((st = resync_launch(L))) return st;
    if (!ba.empty()) {
        hipLaunchKernelGGL(k_branch_batched, dim3((unsigned)ba.size()), dim3(kBranchThreads), 0, stream, dbranch);
        SAIL_HIP(hipGetLastError());
    }
    for (const Launch &L : targets)
        if ((st = resync_launch(L))) return st;
    for (const Launch &L : smooths)
        if ((st = resync_launch(L))) return st;
    if (!bl.empty()) {
        hipLaunchKernelGGL(k_block_record_batched, dim3((unsigned)bl.size()), dim3(kThreads), 0, stream, dblog);
        SAIL_HIP(hipGetLastError());
        for (size_t i = 0; i < act.size(); ++i)
            if (act[i]->p->d_blog && kend[i] % act[i]->sc.resync_every == 0) ++act[i]->p->blog_total;
    }
    SAIL_HIP(hipEventRecord(ring.done[slot], stream));
    for (size_t i = 0; i < act.size(); ++i) act[i]->k = kend[i];
    return SAIL_OK;
}

}  // namespace

#include "arena.h"  // the served loop's arena (host code, tested on the CPU too)

namespace {

// First-fit allocator over one device allocation, with coalescing frees.
using sail_arena::Arena;

enum JobState { kQueued, kRunning, kFinishing, kDone };

struct ServedJob {
    int64_t id = 0;
    std::vector<double> omega, tau, F, sigma, T;
    bool has_sigma = false;
    double m0 = 0, m1 = 0;
    int mode = 0, n_walkers = 0, precision = 0, tpl = 0;
    uint64_t seed = 0;
    sail_schedule sc{};
    size_t need = 0;
    // while admitted
    sail_problem *p = nullptr;
    Region region;
    double *d_mean = nullptr;
    BatchJob bj;
    hipEvent_t done = nullptr;
    bool cancel = false;     // under the server mutex: a running job leaves at the next round boundary
    bool cancelled = false;  // server thread: the job left in flight; its device work is draining
    // outcome
    JobState state = kQueued;
    sail_job_result res{};
    std::vector<double> mean;
};

// Device bytes a served job takes from the arena: the problem at its
// precision, the schedule, a larger event log if needed, the mean-spectrum
// output and alignment.
size_t served_job_bytes(int n_omega, int n_tau, int n_walkers, int precision, int n_T, int branch_every)
{
    size_t b = sail_footprint_bytes(n_omega, n_tau, n_walkers, precision);
    b += sizeof(double) * ((size_t)n_T + (size_t)n_omega);
    const int events = n_T / branch_every + 1;
    if (events > 64) b += (size_t)std::max(events, 128) * (4 * sizeof(double) + 2 * sizeof(int32_t));
    return b + 64 * 256;
}

}  // namespace

struct sail_server {
    int device = 0, max_jobs = 1;
    Arena arena;
    hipStream_t stream = nullptr, setup = nullptr;
    StageRing ring;
    SweepTimer timer;
    std::vector<hipEvent_t> event_pool;
    std::thread thread;
    std::mutex mu;
    std::condition_variable cv_work, cv_done;
    bool stop = false;
    int64_t next_id = 1;
    std::deque<ServedJob *> queue;             // under mu
    std::map<int64_t, ServedJob *> jobs;       // under mu: every job not yet waited for
    std::vector<ServedJob *> active, finishing;  // server thread only
    sail_server_stats stats{};                 // under mu
    std::chrono::steady_clock::time_point t0 = std::chrono::steady_clock::now();
    double now() const { return std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count(); }
};

namespace {

void publish(sail_server *S, ServedJob *j, int status)
{
    std::lock_guard<std::mutex> lk(S->mu);
    j->res.status = status;
    j->res.t_done = S->now();
    j->state = kDone;
    if (status == SAIL_OK) S->stats.completed++;
    else if (status == SAIL_ECANCELLED) S->stats.cancelled++;
    else S->stats.failed++;
    S->stats.arena_used = S->arena.used;
    S->cv_done.notify_all();
}

// Returns the job's device memory to the arena (the device is done with it).
void teardown(sail_server *S, ServedJob *j)
{
    if (j->p) {
        RegionScope rs(&j->region);
        sail_problem_destroy(j->p);
        j->p = nullptr;
    }
    if (j->region.base) S->arena.give(j->region.base, j->need);
    j->region = Region{};
    j->d_mean = nullptr;
    if (j->done) S->event_pool.push_back(j->done);
    j->done = nullptr;
}

sail_status setup_job(sail_server *S, ServedJob *j)
{
    sail_status st;
    int tpl = j->tpl;
    const int No = (int)j->omega.size(), Nt = (int)j->tau.size();
    if (tpl < 0 && !tuned_layout(S->device, No, Nt, j->n_walkers, j->precision, &tpl))
        remember_layout(S->device, No, Nt, j->n_walkers, j->precision, tpl = kDefaultTile, false);
    RegionScope rs(&j->region);
    if ((st = sail_problem_create(j->omega.data(), (int)j->omega.size(), j->tau.data(), (int)j->tau.size(), j->F.data(),
                                  j->has_sigma ? j->sigma.data() : nullptr, j->m0, j->m1, j->mode, S->device, &j->p)))
        return st;
    if ((st = sail_set_tau_per_lane(j->p, tpl < 0 ? 0 : tpl))) return st;
    if ((st = sail_walkers_init(j->p, j->n_walkers, j->seed, j->precision, S->setup))) return st;
    if ((st = check_schedule(j->p, &j->sc, 0, j->sc.n_T))) return st;
    if ((st = prepare_schedule(j->p, &j->sc, j->sc.n_T, S->setup))) return st;
    if ((st = dalloc(&j->d_mean, j->omega.size()))) return st;
    if (S->event_pool.empty()) {
        hipEvent_t e;
        SAIL_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        S->event_pool.push_back(e);
    }
    j->done = S->event_pool.back();
    S->event_pool.pop_back();
    j->bj.p = j->p;
    j->bj.sc = j->sc;
    j->bj.k = 0;
    j->bj.last = j->sc.n_T;
    return SAIL_OK;
}

// Admits queued jobs in arrival order while a slot is free and the head
// job's footprint fits in the arena.
void admit(sail_server *S)
{
    for (;;) {
        ServedJob *j;
        {
            std::lock_guard<std::mutex> lk(S->mu);
            if (S->stop || S->queue.empty() || (int)(S->active.size() + S->finishing.size()) >= S->max_jobs) return;
            j = S->queue.front();
        }
        char *blk = S->arena.take(j->need);
        if (!blk) return;
        {
            std::lock_guard<std::mutex> lk(S->mu);
            S->queue.pop_front();
            S->stats.admitted++;
            S->stats.arena_used = S->arena.used;
            S->stats.arena_peak = S->arena.peak;
            j->state = kRunning;
            j->res.t_admit = S->now();
        }
        j->region = Region{blk, j->need, 0};
        const sail_status st = setup_job(S, j);
        if (st) {
            (void)hipStreamSynchronize(S->setup);
            teardown(S, j);
            publish(S, j, st);
            continue;
        }
        S->active.push_back(j);
    }
}

// Outputs of a finished job, read once its last kernels have completed.
void finalize(sail_server *S, ServedJob *j)
{
    const int No = (int)j->omega.size(), Nw = j->n_walkers;
    std::vector<double> chi2(Nw);
    j->mean.resize(No);
    hipError_t e = hipMemcpy(j->mean.data(), j->d_mean, sizeof(double) * No, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(chi2.data(), j->p->d_chi2, sizeof(double) * Nw, hipMemcpyDeviceToHost);
    int status = e == hipSuccess ? SAIL_OK : SAIL_EDEVICE;
    if (status == SAIL_OK) {
        std::sort(chi2.begin(), chi2.end());
        j->res.chi2_min = chi2[0];
        j->res.chi2_median = (Nw % 2) ? chi2[Nw / 2] : 0.5 * (chi2[Nw / 2 - 1] + chi2[Nw / 2]);
        j->res.chi2_unit = j->p->chi2_unit;
        if (!std::isfinite(j->res.chi2_median)) status = SAIL_ENUMERIC;
    }
    teardown(S, j);
    publish(S, j, status);
}

void serve(sail_server *S)
{
    (void)hipSetDevice(S->device);
    for (;;) {
        for (auto it = S->finishing.begin(); it != S->finishing.end();) {
            const hipError_t q = hipEventQuery((*it)->done);
            if (q == hipErrorNotReady) {
                ++it;
                continue;
            }
            if ((*it)->cancelled) {
                // cancelled in flight: its last kernels are done, so its block can return
                teardown(S, *it);
                publish(S, *it, SAIL_ECANCELLED);
            } else {
                finalize(S, *it);
            }
            it = S->finishing.erase(it);
        }
        (void)S->timer.harvest(false);
        {
            std::lock_guard<std::mutex> lk(S->mu);
            if (S->stop) break;
            S->stats.sweep_ms = S->timer.ms;
            S->stats.sweep_launches = S->timer.n;
        }
        admit(S);
        // cancelled jobs leave between rounds; their block returns once the
        // device has finished the work already enqueued for them
        for (auto it = S->active.begin(); it != S->active.end();) {
            ServedJob *j = *it;
            bool c;
            {
                std::lock_guard<std::mutex> lk(S->mu);
                c = j->cancel;
            }
            if (!c) {
                ++it;
                continue;
            }
            (void)hipEventRecord(j->done, S->stream);
            j->cancelled = true;
            {
                std::lock_guard<std::mutex> lk(S->mu);
                j->state = kFinishing;
            }
            S->finishing.push_back(j);
            it = S->active.erase(it);
        }
        if (!S->active.empty()) {
            std::vector<BatchJob *> bjs;
            for (auto *j : S->active) bjs.push_back(&j->bj);
            sail_status st = batch_round(bjs, S->ring, S->timer, S->stream);
            {
                std::lock_guard<std::mutex> lk(S->mu);
                S->stats.rounds++;
            }
            if (st) {
                (void)hipStreamSynchronize(S->stream);
                for (auto *j : S->active) {
                    teardown(S, j);
                    publish(S, j, st);
                }
                S->active.clear();
                continue;
            }
            for (auto it = S->active.begin(); it != S->active.end();) {
                ServedJob *j = *it;
                if (j->bj.k < j->bj.last) {
                    ++it;
                    continue;
                }
                launch_mean_spectrum(j->n_walkers, (int)j->omega.size(), j->p->d_b, j->p->d_gsc, j->p->d_part, j->d_mean,
                                     S->stream);
                (void)hipEventRecord(j->done, S->stream);
                j->state = kFinishing;
                S->finishing.push_back(j);
                it = S->active.erase(it);
            }
        } else if (!S->finishing.empty()) {
            std::unique_lock<std::mutex> lk(S->mu);
            S->cv_work.wait_for(lk, std::chrono::microseconds(200), [&] { return S->stop; });
        } else {
            std::unique_lock<std::mutex> lk(S->mu);
            S->cv_work.wait(lk, [&] { return S->stop || !S->queue.empty(); });
        }
    }
    // shutdown: let the device finish, then cancel everything still here
    (void)hipStreamSynchronize(S->stream);
    (void)hipStreamSynchronize(S->setup);
    for (auto *j : S->active) {
        teardown(S, j);
        publish(S, j, SAIL_ECANCELLED);
    }
    for (auto *j : S->finishing) {
        teardown(S, j);
        publish(S, j, SAIL_ECANCELLED);
    }
    S->active.clear();
    S->finishing.clear();
    std::lock_guard<std::mutex> lk(S->mu);
    for (auto *j : S->queue) {
        j->res.status = SAIL_ECANCELLED;
        j->res.t_done = S->now();
        j->state = kDone;
        S->stats.cancelled++;
    }
    S->queue.clear();
    S->cv_done.notify_all();
}

}  // namespace

struct sail_batch {
    int device = 0;
    std::vector<sail_problem *> probs;
    StageRing ring;
    SweepTimer timer;
    ~sail_batch() { ring.release(); }
};

extern "C" {

void sail_schedule_defaults(sail_schedule *s)
{
    if (!s) return;
    s->T = nullptr;
    s->n_T = 0;
    s->branch_every = 100;
    s->resync_every = 100;
    s->branch_fraction = 0.25;
    s->imprint_t = 0.1;
    s->eps0 = 0.1;
    s->amp_p = 1.0;
    s->amp_m = 2;
    s->amp_avg = 0.1;
    s->walk_len = 0;
    s->t_units = 0;
    s->smooth = 0.0;
    s->adaptive = 0;
    s->self_cool = 0;
    s->boil_blocks = 0;
    s->cool_blocks = 1;
}

const char *sail_status_string(int status)
{
    switch (status) {
        case SAIL_OK: return "ok";
        case SAIL_EINVAL: return "invalid argument";
        case SAIL_EINFEASIBLE: return "sum rules infeasible";
        case SAIL_ENOMEM: return "out of memory";
        case SAIL_EDEVICE: return "device error";
        case SAIL_ENUMERIC: return "non-finite residue";
        case SAIL_ESTATE: return "call out of order";
        case SAIL_ETIMEOUT: return "timed out";
        case SAIL_ECANCELLED: return "cancelled";
        default: return "unknown status";
    }
}

const char *sail_last_error(void) { return g_err.c_str(); }

sail_status sail_set_allocator(sail_alloc_fn alloc, sail_free_fn release, void *user)
{
    if ((alloc == nullptr) != (release == nullptr)) return fail(SAIL_EINVAL, "give both functions or neither");
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    g_alloc = Allocator{alloc, release, user};
    return SAIL_OK;
}

size_t sail_footprint_bytes(int n_omega, int n_tau, int n_walkers, int precision)
{
    if (n_omega <= 0 || n_tau <= 0 || n_walkers < 0) return 0;
    const size_t rsz = precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t No = (size_t)n_omega, Nw = (size_t)n_walkers;
    // (a walker's coordinates and its share of the read-out's rows: a padded row; and the least of those rows)
    const size_t walkers = sizeof(double) * Nw * (No + 4) + rsz * Nw * max_padding(n_tau, precision) +
                           sizeof(double) * kReadRows * n_tau + sizeof(int32_t) * (3 * Nw + 4) +
                           sizeof(double) * (No + std::max<size_t>(No, 64) + No * (size_t)mean_spans(n_walkers)) + 64 * (4 * sizeof(double) + 2 * sizeof(int32_t)) +
                           sizeof(BranchTree);
    return table_bytes(n_omega, n_tau, precision) + walkers;
}

sail_status sail_problem_create(const double *omega, int n_omega, const double *tau, int n_tau, const double *F,
                                const double *sigma, double m0, double m1, int kernel_mode, int device,
                                sail_problem_t *out)
{
    if (!out) return fail(SAIL_EINVAL, "out is NULL");
    *out = nullptr;
    if (!omega || !tau || !F) return fail(SAIL_EINVAL, "NULL input array");
    if (n_omega < 3 || n_tau < 1) return fail(SAIL_EINVAL, "need n_omega >= 3 and n_tau >= 1");
    if (n_tau > 64 * 16) return fail(SAIL_EINVAL, "n_tau above 1024 is not supported");
    sail_status st;
    if ((st = check_lds(n_omega))) return st;
    if (kernel_mode != SAIL_K_POINT && kernel_mode != SAIL_K_BIN_EXACT) return fail(SAIL_EINVAL, "bad kernel_mode");
    if (!finite_all(omega, n_omega) || !finite_all(tau, n_tau) || !finite_all(F, n_tau))
        return fail(SAIL_EINVAL, "non-finite input");
    if (sigma) {
        if (!finite_all(sigma, n_tau)) return fail(SAIL_EINVAL, "non-finite sigma");
        for (int i = 0; i < n_tau; ++i)
            if (!(sigma[i] > 0.0)) return fail(SAIL_EINVAL, "sigma must be positive");
    }
    for (int i = 0; i < n_tau; ++i)
        if (tau[i] < 0.0) return fail(SAIL_EINVAL, "tau must be non-negative");
    double dw, dt;
    if (!uniform_grid(omega, n_omega, &dw)) return fail(SAIL_EINVAL, "omega grid must be uniform and increasing");
    if (!uniform_grid(tau, n_tau, &dt)) return fail(SAIL_EINVAL, "tau grid must be uniform and increasing");
    if (!(m0 > 0.0) || !std::isfinite(m0) || !std::isfinite(m1)) return fail(SAIL_EINVAL, "bad moments");
    const double mu = m1 / m0;
    if (!(mu > omega[0] && mu < omega[n_omega - 1])) return fail(SAIL_EINFEASIBLE, "m1/m0 outside the frequency window");
    int dev_count = 0;
    if (hipGetDeviceCount(&dev_count) != hipSuccess || device < 0 || device >= dev_count)
        return fail(SAIL_EDEVICE, "no such HIP device");
    SAIL_HIP(hipSetDevice(device));
    int lds_max = 0;
    SAIL_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, device));
    if ((st = check_lds(n_omega, (size_t)lds_max))) return st;

    sail_problem *p = new (std::nothrow) sail_problem();
    if (!p) return fail(SAIL_ENOMEM, "host allocation");
    p->device = device;
    p->n_omega = n_omega;
    p->n_tau = n_tau;
    p->mode = kernel_mode;
    p->dw = dw;
    p->tau0 = tau[0];
    p->dtau = dt;
    p->m0 = m0;
    p->m1 = m1;
    p->A = m0 / dw;
    p->B = m1 / dw;
    p->omega.assign(omega, omega + n_omega);
    p->tau.assign(tau, tau + n_tau);
    p->F.assign(F, F + n_tau);
    p->w.assign(n_tau, 1.0);
    if (sigma)
        for (int i = 0; i < n_tau; ++i) p->w[i] = 1.0 / (sigma[i] * sigma[i]);
    // per-tau factor of the separable kernel
    p->cfac.assign(n_tau, dw / kTwoPi);
    if (kernel_mode == SAIL_K_BIN_EXACT)
        for (int i = 0; i < n_tau; ++i)
            if (tau[i] > 0.0) p->cfac[i] = (std::exp(0.5 * dw * tau[i]) - std::exp(-0.5 * dw * tau[i])) / (kTwoPi * tau[i]);
    if ((st = build_tables(p))) {
        delete p;
        return st;
    }
    if ((st = build_layout(p, SAIL_FP64))) {
        delete p;
        return st;
    }
    if (hipStreamSynchronize(nullptr) != hipSuccess) {  // other streams use them
        delete p;
        return fail(SAIL_EDEVICE, "table kernels failed");
    }
    *out = p;
    return SAIL_OK;
}

void sail_problem_destroy(sail_problem_t p) { delete p; }

sail_status sail_layout(sail_problem_t p, int *lanes_per_walker, int *tau_per_lane)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (lanes_per_walker) *lanes_per_walker = p->lanes;
    if (tau_per_lane) *tau_per_lane = p->tpl;
    return SAIL_OK;
}

sail_status sail_set_tau_per_lane(sail_problem_t p, int tau_per_lane)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (tau_per_lane != 0 && tau_per_lane != 4 && tau_per_lane != 8 && tau_per_lane != 16 && tau_per_lane != 32)
        return fail(SAIL_EINVAL, "tau points per lane must be 0, 4, 8, 16 or 32");
    p->tpl_hint = tau_per_lane;
    return SAIL_OK;
}

// The sweep has one speed and one result whatever the nominal layout, so there is
// nothing to time: the choice is the remembered one (a cache file may hold
// another) or the default tile.
sail_status autotune_layout(sail_problem_t p, int n_walkers, int precision, int *tau_per_lane, void *stream, bool alone)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (precision != SAIL_FP64 && precision != SAIL_FP32) return fail(SAIL_EINVAL, "bad precision");
    if (n_walkers < 2 || n_walkers > kBranchMaxWalkers) return fail(SAIL_EINVAL, "bad walker count");
    int tpl = 0;
    if (!tuned_layout(p->device, p->n_omega, p->n_tau, n_walkers, precision, &tpl, alone)) {
        SAIL_HIP(hipSetDevice(p->device));
        SAIL_HIP(hipStreamSynchronize((hipStream_t)stream));
        p->free_walkers();
        p->chi2_unit = NAN;
        tpl = kDefaultTile;
        remember_layout(p->device, p->n_omega, p->n_tau, n_walkers, precision, tpl, alone);
    }
    p->tpl_hint = tpl;
    if (tau_per_lane) *tau_per_lane = tpl;
    return SAIL_OK;
}

sail_status sail_autotune_layout(sail_problem_t p, int n_walkers, int precision, int *tau_per_lane, void *stream)
{
    return autotune_layout(p, n_walkers, precision, tau_per_lane, stream, false);
}

sail_status sail_autotune_layout_alone(sail_problem_t p, int n_walkers, int precision, int *tau_per_lane,
                                       void *stream)
{
    return autotune_layout(p, n_walkers, precision, tau_per_lane, stream, true);
}

sail_status sail_walkers_init(sail_problem_t p, int n_walkers, uint64_t seed, int precision, void *stream_)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (n_walkers < 2) return fail(SAIL_EINVAL, "need at least two walkers");
    if (precision != SAIL_FP64 && precision != SAIL_FP32) return fail(SAIL_EINVAL, "bad precision");
    if ((size_t)n_walkers * p->n_omega * sizeof(double) >= ((size_t)1 << 31))
        return fail(SAIL_EINVAL, "spectra of all walkers must stay below 2 GiB");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    p->self_T_end = 0;
    std::vector<double> a0;
    sail_status st = start_spectrum(p->omega, p->A, p->B, a0);
    if (st) return st;
    SAIL_HIP(hipStreamSynchronize(stream));
    p->free_walkers();
    if ((st = build_layout(p, precision)) || (st = build_columns(p, precision, stream))) return st;
    const int No = p->n_omega, ntp = p->ntau_pad;
    const size_t rsz = precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t phi_bytes = rsz * (size_t)n_walkers * 4 * p->chunk(precision);
    char *phi = nullptr;
    if ((st = dalloc(&phi, phi_bytes))) return st;
    p->d_phi = phi;
    // rows of the read-out of reconstructions: what the walkers' coordinates
    // leave of a padded row per walker in the loop precision
    const int64_t left = (int64_t)(rsz * (ntp - 4 * p->chunk(precision)));
    p->read_rows = (int)std::max<int64_t>(n_walkers * left / (int64_t)(sizeof(double) * p->n_tau), std::min(n_walkers, kReadRows));
    p->read_rows = std::min(p->read_rows, n_walkers);
    if ((st = dalloc(&p->d_b, (size_t)n_walkers * No)) || (st = dalloc(&p->d_gsc, 2 * (size_t)n_walkers + (size_t)p->read_rows * p->n_tau)) || (st = dalloc(&p->d_ginv, n_walkers)) ||
        (st = dalloc(&p->d_chi2, n_walkers)) || (st = dalloc(&p->d_a0, No)) ||
        (st = dalloc(&p->d_tmp, std::max(No, 64))) || (st = dalloc(&p->d_teff, 1)) ||
        (st = dalloc(&p->d_part, (size_t)mean_spans(n_walkers) * No)) || (st = dalloc(&p->d_m, n_walkers)) || (st = dalloc(&p->d_targets, n_walkers)) ||
        (st = dalloc(&p->d_donors, n_walkers)) || (st = dalloc(&p->d_npairs, 4)) || (st = dalloc(&p->d_tree, 1))) {
        p->free_walkers();
        return st;
    }
    p->d_rate = p->d_gsc + n_walkers;  // one array: what a small population's read-out copies at once
    p->d_F = p->d_rate + n_walkers;
    p->n_walkers = n_walkers;
    p->seed = seed;
    p->precision = precision;
    if ((st = ensure_events(p, 64, stream))) {
        p->free_walkers();
        return st;
    }
    SAIL_HIP(hipMemcpyAsync(p->d_a0, a0.data(), sizeof(double) * No, hipMemcpyHostToDevice, stream));
    SAIL_HIP(hipMemsetAsync(p->d_phi, 0, phi_bytes, stream));  // the padding of the chunks
    SAIL_HIP(hipMemsetAsync(p->d_tree, 0, sizeof(BranchTree), stream));
    const size_t total = (size_t)n_walkers * No;
    hipLaunchKernelGGL(k_init_walkers, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream,
                       n_walkers, No, (const double *)p->d_a0, p->d_b, p->d_gsc, p->d_ginv, p->d_rate);
    SAIL_HIP(hipGetLastError());
    if ((st = launch_resync(p, 0, nullptr, nullptr, n_walkers, stream))) return st;
    double c0 = 0.0;
    SAIL_HIP(hipMemcpyAsync(&c0, p->d_chi2, sizeof(double), hipMemcpyDeviceToHost, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    if (!std::isfinite(c0) || !(c0 > 0.0)) return fail(SAIL_ENUMERIC, "starting residue is not positive and finite");
    p->chi2_unit = c0;
    p->ev_used = 0;
    return SAIL_OK;
}

double sail_chi2_unit(sail_problem_t p) { return p ? p->chi2_unit : NAN; }

sail_status sail_set_event_log(sail_problem_t p, int keep_multipliers)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    SAIL_HIP(hipSetDevice(p->device));
    // the new multiplier log first, so that a failed call leaves the old one
    int32_t *m = nullptr;
    if (keep_multipliers) {
        const size_t n = (size_t)p->cap_events * p->n_walkers;
        sail_status st = dalloc(&m, n);
        if (st) return st;
        const hipError_t e = hipMemset(m, 0, sizeof(int32_t) * std::max<size_t>(n, 1));
        if (e != hipSuccess) {
            dfree(m);
            return fail(SAIL_EDEVICE, std::string("hipMemset: ") + hipGetErrorString(e));
        }
    }
    dfree(p->d_ev_m);
    p->d_ev_m = m;
    p->keep_m = keep_multipliers ? 1 : 0;
    return SAIL_OK;
}

sail_status sail_set_trace(sail_problem_t p, int k0, int k1, double *dchi2, uint8_t *flags)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (k1 < k0 || k0 < 0) return fail(SAIL_EINVAL, "bad trace window");
    if (k1 > k0 && (!dchi2 || !flags)) return fail(SAIL_EINVAL, "trace buffers are NULL");
    p->tk0 = k0;
    p->tk1 = k1;
    p->tr_dchi2 = k1 > k0 ? dchi2 : nullptr;
    p->tr_flags = k1 > k0 ? flags : nullptr;
    return SAIL_OK;
}

sail_status sail_set_timing(sail_problem_t p, int enable)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    p->timing = enable ? 1 : 0;
    p->ev_used = 0;
    return SAIL_OK;
}

sail_status sail_sweep_timing(sail_problem_t p, double *total_ms, int64_t *launches, int reset)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    SAIL_HIP(hipSetDevice(p->device));
    double tot = 0.0;
    for (size_t i = 0; i < p->ev_used; ++i) {
        SAIL_HIP(hipEventSynchronize(p->ev_stop[i]));
        float ms = 0.f;
        SAIL_HIP(hipEventElapsedTime(&ms, p->ev_start[i], p->ev_stop[i]));
        tot += ms;
    }
    if (total_ms) *total_ms = tot;
    if (launches) *launches = (int64_t)p->ev_used;
    if (reset) p->ev_used = 0;
    return SAIL_OK;
}

// Copies the walker state to the watchdog snapshot (to_snapshot; only while
// the flag is clear) or back from it (unconditionally).
sail_status watch_copy(sail_problem *p, bool to_snapshot, hipStream_t stream)
{
    const size_t n = (size_t)p->n_walkers;
    const size_t rsz = p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t phi_words = rsz * n * (size_t)p->phi_row() / sizeof(double);
    struct { double *live, *snap; size_t words; } bufs[] = {
        {p->d_b, p->sn_b, n * (size_t)p->n_omega}, {(double *)p->d_phi, p->sn_phi, phi_words},
        {p->d_gsc, p->sn_gsc, n}, {p->d_ginv, p->sn_ginv, n}, {p->d_chi2, p->sn_chi2, n}, {p->d_rate, p->sn_rate, n}};
    for (auto &bf : bufs) {
        const unsigned grid = (unsigned)std::min<size_t>((bf.words + kThreads - 1) / kThreads, 2048);
        if (to_snapshot)
            hipLaunchKernelGGL(k_watch_copy, dim3(grid), dim3(kThreads), 0, stream, (const unsigned int *)p->d_watch,
                               bf.snap, (const double *)bf.live, bf.words);
        else
            hipLaunchKernelGGL(k_watch_copy, dim3(grid), dim3(kThreads), 0, stream, (const unsigned int *)nullptr,
                               bf.live, (const double *)bf.snap, bf.words);
        SAIL_HIP(hipGetLastError());
    }
    return SAIL_OK;
}

sail_status run_schedule(sail_problem_t p, const sail_schedule *sc, int first_sweep, int n_sweeps, void *stream_)
{
    sail_status st;
    if ((st = check_schedule(p, sc, first_sweep, n_sweeps))) return st;
    if (n_sweeps == 0) return SAIL_OK;
    if (sc->self_cool && first_sweep % sc->branch_every != 0 &&
        !(first_sweep >= p->self_T_k0 && first_sweep < p->self_T_end))
        return fail(SAIL_EINVAL, "a self-cooling run starts at a block boundary or inside the block the previous "
                                 "call on this problem started");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    if ((st = prepare_schedule(p, sc, first_sweep + n_sweeps, stream))) return st;
    const SweepParams sp{sc->eps0, sc->amp_p, sc->amp_avg, sc->amp_m, sc->walk_len};
    const int last = first_sweep + n_sweeps;
    // watchdog: the call's starting state is the first snapshot; every resync
    // checks the walkers, and each clean resync boundary (after its branching
    // event, if any) refreshes the snapshot
    const bool watch = p->watch_bound > 0.0 && p->d_watch;
    struct WatchScope {
        sail_problem *p;
        ~WatchScope() { p->watch_active = false; }
    } watch_scope{p};
    if (watch) {
        p->watch_tripped = p->watch_restored = -1;
        hipLaunchKernelGGL(k_watch_reset, dim3(1), dim3(1), 0, stream, p->d_watch, first_sweep);
        SAIL_HIP(hipGetLastError());
        if ((st = watch_copy(p, true, stream))) return st;
        p->watch_active = true;
    }
    int k = first_sweep;
    while (k < last) {
        if (sc->self_cool && k % sc->branch_every == 0) {
            const int k1 = std::min(k + sc->branch_every, sc->n_T);
            hipLaunchKernelGGL(k_self_cool, dim3(1), dim3(kThreads), 0, stream, (const double *)p->d_chi2, p->n_walkers,
                               k / sc->branch_every, sc->boil_blocks, sc->cool_blocks, p->d_Tabs, k, k1);
            SAIL_HIP(hipGetLastError());
            p->self_T_k0 = k;
            p->self_T_end = k1;
        }
        int kend = segment_end(sc, k, last);
        // split at the trace window edges so untraced sweeps use the fast kernel
        if (p->tk1 > p->tk0) {
            if (k < p->tk0 && kend > p->tk0) kend = p->tk0;
            else if (k < p->tk1 && kend > p->tk1) kend = p->tk1;
        }
        if ((st = launch_sweep(p, k, kend, sp, stream))) return st;
        if (kend % sc->resync_every == 0)
            if ((st = launch_resync(p, 1, nullptr, nullptr, p->n_walkers, stream))) return st;
        if (kend % sc->branch_every == 0) {
            const BranchArgs ba = make_branch_args(p, sc->branch_fraction, kend / sc->branch_every - 1, sc->adaptive,
                                                   sc->imprint_t);
            if ((st = launch_branch(p, ba, stream))) return st;
            if ((st = launch_resync(p, 0, p->d_targets, p->d_npairs, p->n_walkers, stream, p->d_donors, sc->imprint_t,
                                    0.0, sc->adaptive ? p->d_teff : nullptr)))
                return st;
            // Sec. 2.6: every walker smoothed, renormalised and recomputed
            if (sc->smooth > 0.0)
                if ((st = launch_resync(p, 1, nullptr, nullptr, p->n_walkers, stream, nullptr, 0.0, sc->smooth)))
                    return st;
        }
        if (watch && kend % sc->resync_every == 0) {
            if ((st = watch_copy(p, true, stream))) return st;
            hipLaunchKernelGGL(k_watch_mark, dim3(1), dim3(1), 0, stream, p->d_watch, kend);
            SAIL_HIP(hipGetLastError());
        }
        if (p->d_blog && kend % sc->resync_every == 0) {
            const BlockLogArgs bl{p->n_walkers, p->d_chi2, p->d_rate, p->d_drift, p->d_Tabs, kend,
                                  kend % sc->branch_every == 0 ? kend / sc->branch_every - 1 : -1,
                                  p->d_blog + (p->blog_total % p->blog_cap)};
            hipLaunchKernelGGL(k_block_record, dim3(1), dim3(kThreads), 0, stream, bl);
            SAIL_HIP(hipGetLastError());
            ++p->blog_total;
        }
        k = kend;
    }
    if (watch) {
        p->watch_active = false;
        unsigned int w[3] = {0u, 0u, 0u};
        SAIL_HIP(hipMemcpyAsync(w, p->d_watch, sizeof w, hipMemcpyDeviceToHost, stream));
        SAIL_HIP(hipStreamSynchronize(stream));
        if (w[0] != 0u) {
            if ((st = watch_copy(p, false, stream))) return st;
            SAIL_HIP(hipStreamSynchronize(stream));
            p->watch_restored = (int)w[1];
            p->watch_tripped = (int)w[2];
            if (sc->self_cool) {
                // the block holding the restored sweep keeps the temperature it started with
                p->self_T_k0 = (p->watch_restored / sc->branch_every) * sc->branch_every;
                p->self_T_end = std::min(p->self_T_k0 + sc->branch_every, sc->n_T);
            }
            return fail(SAIL_ENUMERIC, std::string("watchdog: ") +
                                           ((w[0] & 2u) ? "a non-finite residue" : "a sum-rule drift above the bound") +
                                           " at the resync after sweep " + std::to_string(p->watch_tripped) +
                                           "; walkers restored to their state at sweep " +
                                           std::to_string(p->watch_restored));
        }
    }
    return SAIL_OK;
}

sail_status sail_run_schedule(sail_problem_t p, const sail_schedule *sc, int first_sweep, int n_sweeps, void *stream_)
{
    const sail_status st = run_schedule(p, sc, first_sweep, n_sweeps, stream_);
    if (p && p->n_walkers > 0) {
        const sail_status sd = mark_done(p, (hipStream_t)stream_);
        if (!st && sd) return sd;
    }
    return st;
}

sail_status sail_set_watchdog(sail_problem_t p, double drift_bound)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (!(drift_bound >= 0.0) || !std::isfinite(drift_bound)) return fail(SAIL_EINVAL, "drift bound must be finite and >= 0");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    SAIL_HIP(hipSetDevice(p->device));
    if (drift_bound == 0.0) {
        p->free_watch();
        return SAIL_OK;
    }
    if (!p->d_watch) {
        const size_t n = (size_t)p->n_walkers;
        const size_t rsz = p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
        sail_status st;
        if ((st = dalloc(&p->d_watch, 4)) || (st = dalloc(&p->sn_b, n * (size_t)p->n_omega)) ||
            (st = dalloc(&p->sn_phi, rsz * n * (size_t)p->phi_row() / sizeof(double))) || (st = dalloc(&p->sn_gsc, n)) ||
            (st = dalloc(&p->sn_ginv, n)) || (st = dalloc(&p->sn_chi2, n)) || (st = dalloc(&p->sn_rate, n))) {
            p->free_watch();
            return st;
        }
    }
    p->watch_bound = drift_bound;
    p->watch_tripped = p->watch_restored = -1;
    return SAIL_OK;
}

sail_status sail_set_block_log(sail_problem_t p, int capacity)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (capacity < 0) return fail(SAIL_EINVAL, "capacity must be >= 0");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    SAIL_HIP(hipSetDevice(p->device));
    // the new ring first, so that a failed allocation leaves the old log as it was
    sail_block_record *ring = nullptr;
    double *drift = nullptr;
    if (capacity > 0) {
        sail_status st;
        if ((st = dalloc(&ring, (size_t)capacity)) || (st = dalloc(&drift, (size_t)p->n_walkers))) {
            dfree(ring);
            dfree(drift);
            return st;
        }
    }
    p->free_block_log();
    p->d_blog = ring;
    p->d_drift = drift;
    p->blog_cap = capacity;
    return SAIL_OK;
}

sail_status sail_read_block_log(sail_problem_t p, sail_block_record *out, int max_records, int *n_records,
                                int64_t *n_total, void *stream_)
{
    if (!p || (!out && max_records > 0)) return fail(SAIL_EINVAL, "NULL argument");
    if (max_records < 0) return fail(SAIL_EINVAL, "max_records must be >= 0");
    if (!p->d_blog) return fail(SAIL_ESTATE, "the block log is off (sail_set_block_log)");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    const int64_t held = std::min<int64_t>(p->blog_total, p->blog_cap);
    const int n = (int)std::min<int64_t>(held, max_records);
    // the newest n records, oldest first; the ring may wrap once
    const int64_t first = p->blog_total - n;
    const int s0 = (int)(first % p->blog_cap);
    const int part = std::min(n, p->blog_cap - s0);
    if (part > 0)
        SAIL_HIP(hipMemcpyAsync(out, p->d_blog + s0, sizeof(sail_block_record) * part, hipMemcpyDeviceToHost, stream));
    if (n > part)
        SAIL_HIP(hipMemcpyAsync(out + part, p->d_blog, sizeof(sail_block_record) * (n - part), hipMemcpyDeviceToHost,
                                stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    if (n_records) *n_records = n;
    if (n_total) *n_total = p->blog_total;
    return SAIL_OK;
}

sail_status sail_watchdog_report(sail_problem_t p, int *tripped_after_sweep, int *restored_to_sweep)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (tripped_after_sweep) *tripped_after_sweep = p->watch_tripped;
    if (restored_to_sweep) *restored_to_sweep = p->watch_restored;
    return SAIL_OK;
}

sail_status sail_read_chi2(sail_problem_t p, double *out, void *stream_)
{
    if (!p || !out) return fail(SAIL_EINVAL, "NULL argument");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    SAIL_HIP(hipMemcpyAsync(out, p->d_chi2, sizeof(double) * p->n_walkers, hipMemcpyDeviceToHost, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    return SAIL_OK;
}

sail_status sail_read_spectrum(sail_problem_t p, double *out, void *stream_)
{
    if (!p || !out) return fail(SAIL_EINVAL, "NULL argument");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    std::lock_guard<std::mutex> lock(p->read_mu);
    // d_tmp holds max(64, n_omega) doubles (allocated with the walkers)
    launch_mean_spectrum(p->n_walkers, p->n_omega, p->d_b, p->d_gsc, p->d_part, p->d_tmp, stream);
    SAIL_HIP(hipGetLastError());
    SAIL_HIP(hipMemcpyAsync(out, p->d_tmp, sizeof(double) * p->n_omega, hipMemcpyDeviceToHost, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    return SAIL_OK;
}

sail_status sail_read_chi2_hist_noalloc(sail_problem_t p, int n_bins, double lo, double hi, uint64_t *counts,
                                        void *stream_)
{
    if (!p || !counts) return fail(SAIL_EINVAL, "NULL argument");
    if (n_bins <= 0 || n_bins > kNoAllocMaxBins)
        return fail(SAIL_EINVAL, "n_bins must lie in [1, " + std::to_string(kNoAllocMaxBins) +
                                     "] (the size of the device-resident scratch)");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    unsigned long long *sc = nullptr;
    sail_status st = scratch_of_device(p->device, &sc);
    if (st) return st;
    double *range = (double *)sc;
    unsigned long long *d_counts = sc + kScratchRangeWords;
    SAIL_HIP(launch_chi2_hist(p->n_walkers, p->d_chi2, n_bins, lo, hi, range, d_counts, stream));
    SAIL_HIP(hipMemcpyAsync(counts, d_counts, sizeof(uint64_t) * n_bins, hipMemcpyDefault, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    return SAIL_OK;
}

sail_status sail_read_chi2_hist(sail_problem_t p, int n_bins, double lo, double hi, uint64_t *counts, void *stream_)
{
    if (!p || !counts || n_bins <= 0 || n_bins > 4096) return fail(SAIL_EINVAL, "bad histogram arguments");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    std::lock_guard<std::mutex> lock(p->read_mu);
    if (n_bins > p->cap_hist) {
        unsigned long long *d = nullptr;
        const sail_status st = dalloc(&d, n_bins);
        if (st) return st;
        dfree(p->d_hist);
        p->d_hist = d;
        p->cap_hist = n_bins;
    }
    SAIL_HIP(launch_chi2_hist(p->n_walkers, p->d_chi2, n_bins, lo, hi, p->d_tmp, p->d_hist, stream));
    SAIL_HIP(hipMemcpyAsync(counts, p->d_hist, sizeof(uint64_t) * n_bins, hipMemcpyDeviceToHost, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    return SAIL_OK;
}

sail_status sail_read_state(sail_problem_t p, double *a, double *F, double *rate, void *stream_)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    const int n = p->n_walkers, No = p->n_omega, Nt = p->n_tau;
    std::unique_lock<std::mutex> rows_lock(p->read_mu, std::defer_lock);
    if (F) rows_lock.lock();
    auto reconstruct = [&](int l) {
        const int rows = std::min(p->read_rows, n - l), wpb = resync_wpb(No, rows);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(resync_blocks(rows, wpb)), dim3(kThreads), resync_shmem(No, wpb), stream, rows, No, Nt,
                               p->cols(), (const double *)p->d_E, (const double *)p->d_cfac,
                               (const double *)p->d_b + (size_t)l * No, (const double *)p->d_gsc + l, p->d_F);
        };
        if (p->precision == SAIL_FP32) wpb == 16 ? launch(k_reconstruct<float, 16>) : launch(k_reconstruct<float, 8>);
        else wpb == 16 ? launch(k_reconstruct<double, 16>) : launch(k_reconstruct<double, 8>);
        return hipGetLastError();
    };
    // Small populations: scales, rates and reconstructions in one copy (64
    // walkers, 64 bins, 32 times: 82 us in all, most of it the copies)
    const bool once = F && p->read_rows >= n && (size_t)n * Nt <= 65536;
    if (once) SAIL_HIP(reconstruct(0));
    std::vector<double> g(2 * (size_t)n + (once ? (size_t)n * Nt : 0));
    if (a) SAIL_HIP(hipMemcpyAsync(a, p->d_b, sizeof(double) * (size_t)n * No, hipMemcpyDeviceToHost, stream));
    if (a || rate || once) SAIL_HIP(hipMemcpyAsync(g.data(), p->d_gsc, sizeof(double) * g.size(), hipMemcpyDeviceToHost, stream));
    SAIL_HIP(hipStreamSynchronize(stream));
    // (the first rows are computed while the host scales the spectra)
    if (F && !once) SAIL_HIP(reconstruct(0));
    if (rate) std::copy(g.begin() + n, g.begin() + 2 * n, rate);
    if (once) std::copy(g.begin() + 2 * n, g.end(), F);
    if (a)
        for (int l = 0; l < n; ++l)
            for (int j = 0; j < No; ++j) a[(size_t)l * No + j] = g[l] * a[(size_t)l * No + j];
    for (int l = 0; F && !once && l < n; l += p->read_rows) {
        if (l > 0) SAIL_HIP(reconstruct(l));
        SAIL_HIP(hipMemcpyAsync(F + (size_t)l * Nt, p->d_F, sizeof(double) * (size_t)std::min(p->read_rows, n - l) * Nt,
                                hipMemcpyDeviceToHost, stream));
    }
    if (F && !once) SAIL_HIP(hipStreamSynchronize(stream));
    return SAIL_OK;
}

sail_status sail_read_events(sail_problem_t p, int n_events, double *delta, double *pr, int32_t *z, int32_t *status,
                             int32_t *m)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (n_events < 0 || n_events > p->cap_events) return fail(SAIL_EINVAL, "event range outside the log");
    if (m && !p->keep_m) return fail(SAIL_ESTATE, "multipliers were not logged");
    SAIL_HIP(hipSetDevice(p->device));
    if (n_events == 0) return SAIL_OK;
    // the log is written on whatever stream the anneal ran on: a private stream
    // waits for the last recorded anneal work and carries the copies
    if (!p->read_stream) SAIL_HIP(hipStreamCreateWithFlags(&p->read_stream, hipStreamNonBlocking));
    hipStream_t rs = p->read_stream;
    if (p->done_ev) SAIL_HIP(hipStreamWaitEvent(rs, p->done_ev, 0));
    if (delta) SAIL_HIP(hipMemcpyAsync(delta, p->d_ev_delta, sizeof(double) * n_events, hipMemcpyDeviceToHost, rs));
    if (pr) SAIL_HIP(hipMemcpyAsync(pr, p->d_ev_pr, sizeof(double) * n_events, hipMemcpyDeviceToHost, rs));
    if (z) SAIL_HIP(hipMemcpyAsync(z, p->d_ev_z, sizeof(int32_t) * n_events, hipMemcpyDeviceToHost, rs));
    if (status) SAIL_HIP(hipMemcpyAsync(status, p->d_ev_status, sizeof(int32_t) * n_events, hipMemcpyDeviceToHost, rs));
    if (m)
        SAIL_HIP(hipMemcpyAsync(m, p->d_ev_m, sizeof(int32_t) * (size_t)n_events * p->n_walkers, hipMemcpyDeviceToHost,
                                rs));
    SAIL_HIP(hipStreamSynchronize(rs));
    return SAIL_OK;
}

sail_status sail_read_event_margins(sail_problem_t p, int n_events, double *gap, double *bracket)
{
    if (!p) return fail(SAIL_EINVAL, "NULL problem");
    if (n_events < 0 || n_events > p->cap_events) return fail(SAIL_EINVAL, "event range outside the log");
    SAIL_HIP(hipSetDevice(p->device));
    if (n_events == 0) return SAIL_OK;
    if (!p->read_stream) SAIL_HIP(hipStreamCreateWithFlags(&p->read_stream, hipStreamNonBlocking));
    hipStream_t rs = p->read_stream;
    if (p->done_ev) SAIL_HIP(hipStreamWaitEvent(rs, p->done_ev, 0));
    if (gap) SAIL_HIP(hipMemcpyAsync(gap, p->d_ev_gap, sizeof(double) * n_events, hipMemcpyDeviceToHost, rs));
    if (bracket)
        SAIL_HIP(hipMemcpyAsync(bracket, p->d_ev_bracket, sizeof(double) * n_events, hipMemcpyDeviceToHost, rs));
    SAIL_HIP(hipStreamSynchronize(rs));
    return SAIL_OK;
}

// Checkpoint layout: header, then b [N_w][N_omega], phi [N_w][phi_row] in the
// loop precision, g, 1/g, chi^2, rate [N_w], and the digest of the basis that
// phi is in, all little-endian as in memory.  phi means something in that basis
// alone, which follows from the weights and the times (and the selection's
// rounding): coordinates in another one, as of a problem with other errors, are
// not read, and those of version 4, which had no digest, neither.  Version 3 held
// the reconstructions Phi [N_w][ntau_pad] in place of phi (phi_row 0).  Where phi
// is not read it is taken from the spectra, with the residues.
struct StateHeader {
    uint64_t magic;  // "SALIStv5"
    int32_t n_walkers, n_omega, n_tau, ntau_pad, precision, phi_row;
    uint64_t seed;
    double chi2_unit;
};
constexpr uint64_t kStateMagic = 0x35767453494c4153ull, kStateMagicV4 = 0x34767453494c4153ull,
                   kStateMagicV3 = 0x33767453494c4153ull;

// (version 3 and 4 files end before the digest)
size_t state_bytes(const sail_problem *p, int row, bool digest = true)
{
    const size_t n = (size_t)p->n_walkers, rsz = p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    return sizeof(StateHeader) + sizeof(double) * n * p->n_omega + rsz * n * row + 4 * sizeof(double) * n +
           (digest ? sizeof(uint64_t) : 0);
}

sail_status sail_state_export(sail_problem_t p, void *buf, size_t *bytes, void *stream_)
{
    if (!p || !bytes) return fail(SAIL_EINVAL, "NULL argument");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers first");
    const size_t need = state_bytes(p, p->phi_row());
    if (!buf) {
        *bytes = need;
        return SAIL_OK;
    }
    if (*bytes < need) return fail(SAIL_EINVAL, "buffer too small");
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    StateHeader h{kStateMagic, p->n_walkers, p->n_omega, p->n_tau, p->ntau_pad, p->precision, p->phi_row(), p->seed, p->chi2_unit};
    char *o = (char *)buf;
    std::memcpy(o, &h, sizeof h);
    o += sizeof h;
    const size_t n = (size_t)p->n_walkers, rsz = p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t sb = sizeof(double) * n * p->n_omega, sp = rsz * n * p->phi_row(), sv = sizeof(double) * n;
    SAIL_HIP(hipMemcpyAsync(o, p->d_b, sb, hipMemcpyDeviceToHost, stream));
    o += sb;
    SAIL_HIP(hipMemcpyAsync(o, p->d_phi, sp, hipMemcpyDeviceToHost, stream));
    o += sp;
    SAIL_HIP(hipMemcpyAsync(o, p->d_gsc, sv, hipMemcpyDeviceToHost, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(o, p->d_ginv, sv, hipMemcpyDeviceToHost, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(o, p->d_chi2, sv, hipMemcpyDeviceToHost, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(o, p->d_rate, sv, hipMemcpyDeviceToHost, stream));
    o += sv;
    std::memcpy(o, &p->basis_id, sizeof p->basis_id);
    SAIL_HIP(hipStreamSynchronize(stream));
    *bytes = need;
    return SAIL_OK;
}

sail_status sail_state_import(sail_problem_t p, const void *buf, size_t bytes, void *stream_)
{
    if (!p || !buf) return fail(SAIL_EINVAL, "NULL argument");
    if (p->n_walkers == 0) return fail(SAIL_ESTATE, "initialise walkers with the checkpoint's count and precision first");
    StateHeader h;
    if (bytes < sizeof h) return fail(SAIL_EINVAL, "checkpoint truncated");
    std::memcpy(&h, buf, sizeof h);
    const bool v3 = h.magic == kStateMagicV3, digest = h.magic == kStateMagic;
    if (!digest && !v3 && h.magic != kStateMagicV4) return fail(SAIL_EINVAL, "not a checkpoint");
    // (phi does not depend on the padding of the times: only version 3's rows do)
    const int row = v3 ? h.ntau_pad : h.phi_row;
    if (h.n_walkers != p->n_walkers || h.n_omega != p->n_omega || h.n_tau != p->n_tau || (v3 && h.ntau_pad != p->ntau_pad) ||
        h.precision != p->precision || row <= 0)
        return fail(SAIL_EINVAL, "checkpoint does not match this problem's shape, layout or precision");
    const size_t need = state_bytes(p, row, digest);
    if (bytes < need) return fail(SAIL_EINVAL, "checkpoint truncated");
    uint64_t id = 0;
    if (digest) std::memcpy(&id, (const char *)buf + need - sizeof id, sizeof id);
    const bool same_basis = digest && id == p->basis_id && row == p->phi_row();
    p->self_T_end = 0;
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(p->device));
    const char *o = (const char *)buf + sizeof h;
    const size_t n = (size_t)p->n_walkers, rsz = p->precision == SAIL_FP32 ? sizeof(float) : sizeof(double);
    const size_t sb = sizeof(double) * n * p->n_omega, sp = rsz * n * row, sv = sizeof(double) * n;
    SAIL_HIP(hipMemcpyAsync(p->d_b, o, sb, hipMemcpyHostToDevice, stream));
    o += sb;
    if (same_basis) SAIL_HIP(hipMemcpyAsync(p->d_phi, o, sp, hipMemcpyHostToDevice, stream));
    o += sp;
    SAIL_HIP(hipMemcpyAsync(p->d_gsc, o, sv, hipMemcpyHostToDevice, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(p->d_ginv, o, sv, hipMemcpyHostToDevice, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(p->d_chi2, o, sv, hipMemcpyHostToDevice, stream));
    o += sv;
    SAIL_HIP(hipMemcpyAsync(p->d_rate, o, sv, hipMemcpyHostToDevice, stream));
    if (!same_basis) {
        const sail_status st = launch_resync(p, 0, nullptr, nullptr, p->n_walkers, stream);
        if (st) return st;
    }
    SAIL_HIP(hipStreamSynchronize(stream));
    p->seed = h.seed;
    p->chi2_unit = h.chi2_unit;
    return SAIL_OK;
}

// --------------------------------------------------------------------------
// Batches
// --------------------------------------------------------------------------
sail_status sail_batch_create(const sail_problem_t *problems, int n_problems, sail_batch_t *out)
{
    if (!problems || !out || n_problems <= 0) return fail(SAIL_EINVAL, "bad batch arguments");
    *out = nullptr;
    for (int i = 0; i < n_problems; ++i) {
        if (!problems[i]) return fail(SAIL_EINVAL, "NULL problem in batch");
        if (problems[i]->device != problems[0]->device) return fail(SAIL_EINVAL, "batch problems live on different devices");
        for (int j = 0; j < i; ++j)
            if (problems[j] == problems[i]) return fail(SAIL_EINVAL, "a problem appears twice in the batch");
    }
    sail_batch *b = new (std::nothrow) sail_batch;
    if (!b) return fail(SAIL_ENOMEM, "batch");
    b->device = problems[0]->device;
    b->probs.assign(problems, problems + n_problems);
    *out = b;
    return SAIL_OK;
}

void sail_batch_destroy(sail_batch_t b)
{
    if (!b) return;
    (void)hipSetDevice(b->device);
    delete b;
}

sail_status sail_batch_run(sail_batch_t b, const sail_schedule *const *scheds, const int *first_sweep,
                           const int *n_sweeps, void *stream_)
{
    if (!b || !scheds || !first_sweep || !n_sweeps) return fail(SAIL_EINVAL, "NULL argument");
    const int n = (int)b->probs.size();
    sail_status st = SAIL_OK;
    for (int i = 0; i < n; ++i) {
        sail_problem *p = b->probs[i];
        if ((st = check_schedule(p, scheds[i], first_sweep[i], n_sweeps[i]))) return st;
        if (p->precision == SAIL_FP32 ? (p->tpl != 8 && p->tpl != 16 && p->tpl != 32)
                                      : (p->tpl != 4 && p->tpl != 8 && p->tpl != 16))
            return fail(SAIL_EINVAL, "unsupported tau points per lane");
        if (p->tk1 > p->tk0 && first_sweep[i] < p->tk1 && first_sweep[i] + n_sweeps[i] > p->tk0 &&
            scheds[i]->walk_len > 0)
            return fail(SAIL_EINVAL, "traced sweeps of a batch take uniform index selection (walk_len 0)");
        if (scheds[i]->self_cool && first_sweep[i] % scheds[i]->branch_every != 0 &&
            !(first_sweep[i] >= p->self_T_k0 && first_sweep[i] < p->self_T_end))
            return fail(SAIL_EINVAL, "a self-cooling run starts at a block boundary or inside the block the previous "
                                     "call on this problem started");
    }
    hipStream_t stream = (hipStream_t)stream_;
    SAIL_HIP(hipSetDevice(b->device));
    std::vector<BatchJob> jobs(n);
    std::vector<BatchJob *> ptrs;
    for (int i = 0; i < n; ++i) {
        if ((st = prepare_schedule(b->probs[i], scheds[i], first_sweep[i] + n_sweeps[i], stream))) return st;
        jobs[i].p = b->probs[i];
        jobs[i].sc = *scheds[i];
        jobs[i].k = first_sweep[i];
        jobs[i].last = first_sweep[i] + n_sweeps[i];
        ptrs.push_back(&jobs[i]);
    }
    for (;;) {
        bool any = false;
        for (auto *j : ptrs) any = any || j->k < j->last;
        if (!any) break;
        if ((st = batch_round(ptrs, b->ring, b->timer, stream))) break;
    }
    for (int i = 0; i < n; ++i) {
        const sail_status sd = mark_done(b->probs[i], stream);
        if (!st) st = sd;
    }
    return st;
}

sail_status sail_batch_set_timing(sail_batch_t b, int enable)
{
    if (!b) return fail(SAIL_EINVAL, "NULL batch");
    b->timer.enabled = enable != 0;
    return SAIL_OK;
}

sail_status sail_batch_sweep_timing(sail_batch_t b, double *total_ms, int64_t *launches, int reset)
{
    if (!b) return fail(SAIL_EINVAL, "NULL batch");
    SAIL_HIP(hipSetDevice(b->device));
    return b->timer.total(total_ms, launches, reset != 0);
}

// --------------------------------------------------------------------------
// Server
// --------------------------------------------------------------------------
sail_status sail_server_create(const sail_server_config *cfg, sail_server_t *out)
{
    if (!cfg || !out) return fail(SAIL_EINVAL, "NULL argument");
    *out = nullptr;
    if (cfg->max_jobs < 1 || cfg->hbm_bytes < ((size_t)1 << 20)) return fail(SAIL_EINVAL, "bad server configuration");
    int dev_count = 0;
    if (hipGetDeviceCount(&dev_count) != hipSuccess || cfg->device < 0 || cfg->device >= dev_count)
        return fail(SAIL_EDEVICE, "no such HIP device");
    SAIL_HIP(hipSetDevice(cfg->device));
    sail_server *S = new (std::nothrow) sail_server;
    if (!S) return fail(SAIL_ENOMEM, "server");
    S->device = cfg->device;
    S->max_jobs = cfg->max_jobs;
    const size_t bytes = Arena::round_up(cfg->hbm_bytes);
    if (raw_alloc((void **)&S->arena.base, bytes) != hipSuccess) {
        delete S;
        return fail(SAIL_ENOMEM, "server arena");
    }
    S->arena.size = bytes;
    S->arena.free_[0] = bytes;
    if (hipStreamCreateWithFlags(&S->stream, hipStreamNonBlocking) != hipSuccess ||
        hipStreamCreateWithFlags(&S->setup, hipStreamNonBlocking) != hipSuccess) {
        if (S->stream) (void)hipStreamDestroy(S->stream);
        raw_free(S->arena.base);
        delete S;
        return fail(SAIL_EDEVICE, "server streams");
    }
    sail_status st = S->ring.reserve(S->max_jobs);
    if (st) {
        (void)hipStreamDestroy(S->stream);
        (void)hipStreamDestroy(S->setup);
        raw_free(S->arena.base);
        delete S;
        return st;
    }
    S->timer.enabled = 1;
    S->stats.arena_bytes = bytes;
    S->thread = std::thread(serve, S);
    *out = S;
    return SAIL_OK;
}

sail_status sail_server_submit(sail_server_t S, const sail_job *job, int64_t *id)
{
    if (!S || !job || !id) return fail(SAIL_EINVAL, "NULL argument");
    if (!job->omega || !job->tau || !job->F) return fail(SAIL_EINVAL, "NULL input array");
    if (job->n_omega < 3 || job->n_tau < 1) return fail(SAIL_EINVAL, "need n_omega >= 3 and n_tau >= 1");
    if (job->n_tau > 64 * 16) return fail(SAIL_EINVAL, "n_tau above 1024 is not supported");
    sail_status st;
    if ((st = check_lds(job->n_omega))) return st;
    if (job->n_walkers < 2 || job->n_walkers > kBranchMaxWalkers) return fail(SAIL_EINVAL, "bad walker count");
    if (job->precision != SAIL_FP64 && job->precision != SAIL_FP32) return fail(SAIL_EINVAL, "bad precision");
    if (job->tau_per_lane != -1 && job->tau_per_lane != 0 && job->tau_per_lane != 4 && job->tau_per_lane != 8 &&
        job->tau_per_lane != 16 && job->tau_per_lane != 32)
        return fail(SAIL_EINVAL, "bad tau points per lane");
    if ((st = check_schedule_params(&job->sched, 0, job->sched.n_T))) return st;

    ServedJob *j = new (std::nothrow) ServedJob;
    if (!j) return fail(SAIL_ENOMEM, "job");
    j->omega.assign(job->omega, job->omega + job->n_omega);
    j->tau.assign(job->tau, job->tau + job->n_tau);
    j->F.assign(job->F, job->F + job->n_tau);
    j->has_sigma = job->sigma != nullptr;
    if (j->has_sigma) j->sigma.assign(job->sigma, job->sigma + job->n_tau);
    j->T.assign(job->sched.T, job->sched.T + job->sched.n_T);
    j->m0 = job->m0;
    j->m1 = job->m1;
    j->mode = job->kernel_mode;
    j->n_walkers = job->n_walkers;
    j->precision = job->precision;
    j->tpl = job->tau_per_lane;
    j->seed = job->seed;
    j->sc = job->sched;
    j->sc.T = j->T.data();
    j->need = served_job_bytes(job->n_omega, job->n_tau, job->n_walkers, job->precision, job->sched.n_T,
                               job->sched.branch_every);
    j->res.n_omega = job->n_omega;
    j->res.n_walkers = job->n_walkers;
    if (Arena::round_up(j->need) > S->arena.size) {
        delete j;
        return fail(SAIL_EINVAL, "job footprint exceeds the server arena");
    }
    {
        std::lock_guard<std::mutex> lk(S->mu);
        if (S->stop) {
            delete j;
            return fail(SAIL_ESTATE, "server is shutting down");
        }
        j->id = S->next_id++;
        j->res.t_submit = S->now();
        S->jobs[j->id] = j;
        S->queue.push_back(j);
        S->stats.submitted++;
        *id = j->id;
    }
    S->cv_work.notify_one();
    return SAIL_OK;
}

sail_status sail_server_wait(sail_server_t S, int64_t id, double timeout_s, sail_job_result *res, double *mean_spectrum)
{
    if (!S || !res) return fail(SAIL_EINVAL, "NULL argument");
    std::unique_lock<std::mutex> lk(S->mu);
    auto done = [&] {
        auto it = S->jobs.find(id);
        return it == S->jobs.end() || it->second->state == kDone;
    };
    if (timeout_s < 0) S->cv_done.wait(lk, done);
    else if (!S->cv_done.wait_for(lk, std::chrono::duration<double>(timeout_s), done))
        return fail(SAIL_ETIMEOUT, "job still running");
    auto it = S->jobs.find(id);
    if (it == S->jobs.end()) return fail(SAIL_EINVAL, "unknown job id");
    ServedJob *j = it->second;
    *res = j->res;
    if (mean_spectrum && j->res.status == SAIL_OK) std::copy(j->mean.begin(), j->mean.end(), mean_spectrum);
    S->jobs.erase(it);
    delete j;
    return SAIL_OK;
}

sail_status sail_server_get_stats(sail_server_t S, sail_server_stats *out)
{
    if (!S || !out) return fail(SAIL_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lk(S->mu);
    *out = S->stats;
    out->queued = (int)S->queue.size();
    int in_flight = 0;
    for (auto &kv : S->jobs)
        if (kv.second->state == kRunning || kv.second->state == kFinishing) in_flight++;
    out->in_flight = in_flight;
    return SAIL_OK;
}

double sail_server_clock(sail_server_t S) { return S ? S->now() : NAN; }

size_t sail_job_footprint_bytes(const sail_job *job)
{
    if (!job || job->n_omega <= 0 || job->n_tau <= 0 || job->n_walkers < 0 || job->sched.n_T <= 0 ||
        job->sched.branch_every <= 0)
        return 0;
    if (check_schedule_params(&job->sched, 0, job->sched.n_T) != SAIL_OK) return 0;
    return Arena::round_up(served_job_bytes(job->n_omega, job->n_tau, job->n_walkers, job->precision, job->sched.n_T,
                                            job->sched.branch_every));
}

sail_status sail_server_poll(sail_server_t S, int64_t id, int *state)
{
    if (!S || !state) return fail(SAIL_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lk(S->mu);
    auto it = S->jobs.find(id);
    if (it == S->jobs.end()) return fail(SAIL_EINVAL, "unknown job id");
    const JobState js = it->second->state;
    *state = js == kQueued ? SAIL_JOB_QUEUED : js == kDone ? SAIL_JOB_DONE : SAIL_JOB_RUNNING;
    return SAIL_OK;
}

sail_status sail_server_cancel(sail_server_t S, int64_t id)
{
    if (!S) return fail(SAIL_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lk(S->mu);
    auto it = S->jobs.find(id);
    if (it == S->jobs.end()) return fail(SAIL_EINVAL, "unknown job id");
    ServedJob *j = it->second;
    if (j->state == kQueued) {
        S->queue.erase(std::find(S->queue.begin(), S->queue.end(), j));
        j->res.status = SAIL_ECANCELLED;
        j->res.t_done = S->now();
        j->state = kDone;
        S->stats.cancelled++;
        S->cv_done.notify_all();
        return SAIL_OK;
    }
    if (j->state == kRunning) {
        if (!j->cancel) {
            j->cancel = true;
            S->cv_work.notify_all();
        }
        return SAIL_OK;
    }
    return fail(SAIL_ESTATE, "the job has already finished its anneal");
}

void sail_server_destroy(sail_server_t S)
{
    if (!S) return;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        S->stop = true;
    }
    S->cv_work.notify_all();
    if (S->thread.joinable()) S->thread.join();
    (void)hipSetDevice(S->device);
    for (auto &kv : S->jobs) delete kv.second;
    S->jobs.clear();
    S->ring.release();
    for (auto e : S->event_pool) (void)hipEventDestroy(e);
    if (S->stream) (void)hipStreamDestroy(S->stream);
    if (S->setup) (void)hipStreamDestroy(S->setup);
    if (S->arena.base) raw_free(S->arena.base);
    delete S;
}

}  // extern "C"

