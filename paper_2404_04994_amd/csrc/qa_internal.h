// qa_internal.h -- device-side records and launch wrappers of libqarray.
//
// Layout in HBM (one call = one diagram unless batched):
//   DiagRec  : per diagram, written by the prologue kernel (k_prep):
//              C_dd, A = C_dd^{-1} (FP64, symmetric), C_gd, C_dd 1, sums,
//              and the FP32 / split-BF16 tables the matrix-core scorer reads.
//   PixRec   : per pixel, written by the setup kernel (k_setup):
//              the candidate description (n0, free mask, k) and the FP64
//              gradient g0 = A (n0 - x_u) and energy U(n0) at the base state.
//   SavedRec : per pixel, the softargmin state the adjoint needs (the
//              caller-owned "saved" buffer of qa_soft_charge): candidate
//              set, smallest energy, normaliser and mean offset; no energies.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace qa {

constexpr int kMaxDot = 16;
constexpr int kMaxGate = 32;
constexpr int kWave = 64;

// counters (int64) kept in the workspace, mirrored into qa_stats.  Atomics
// on one address from every block serialise at the memory side, so the
// statistics are spread over kCounterSlots cache lines ([slot][C_NUM], a
// block adds to slot blockIdx mod kCounterSlots) and summed by the host.
constexpr int kCounterSlots = 64;
enum Counter {
    C_PIXELS = 0,
    C_QP = 1,
    C_QP_FAIL = 2,
    C_DOUBLED = 3,
    C_NEAR_TIE = 4,
    C_GAP_1E9 = 5,
    C_CANDIDATES = 6,
    C_SCORED = 7,       // states whose approximate energy a scorer computed
    C_UNUSED8 = 8,
    C_UNUSED9 = 9,
    C_NUM = 16
};
constexpr int kCounterWords = kCounterSlots * C_NUM;

// add a block's partial count to its counter slot
__device__ __forceinline__ void block_add_counter(int64_t *counters, int which, int64_t v)
{
    if (v)
        atomicAdd((unsigned long long *)&counters[(blockIdx.x & (kCounterSlots - 1)) * C_NUM + which],
                  (unsigned long long)v);
}

// Cross-lane all-reductions without LDS: DPP within each 16-lane row
// (exchange with lane ^ 1, lane ^ 2, then the mirror images within 8 and 16
// lanes, each an involution, so after four steps every lane of a row holds
// the row's result), then the row swaps of gfx950 for 16 and 32 lanes.
// Every pattern used here (quad permutations, row mirrors, row broadcasts) has
// a valid source lane for every lane, so the move needs no "old" value: the
// plain DPP move, not the update form, whose old operand costs a v_mov per
// use.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
// lane i of every 16-lane row to the whole row
constexpr int kDppRowBcast0 = 0x150;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dppf(float x)
{
    return __uint_as_float(dpp32<CTRL>(__float_as_uint(x)));
}
template <int CTRL>
__device__ __forceinline__ double dppd(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    if constexpr (CTRL >= kDppRowBcast0 && CTRL < kDppRowBcast0 + 16) {
        // (a row broadcast moves both halves at once)
        return __longlong_as_double(
            __builtin_amdgcn_mov_dpp((long long)u, CTRL, 0xF, 0xF, true));
    } else {
        const uint64_t r = (uint64_t)dpp32<CTRL>((uint32_t)u) |
                           ((uint64_t)dpp32<CTRL>((uint32_t)(u >> 32)) << 32);
        return __longlong_as_double((long long)r);
    }
}

// acc + sum_q t_q x(lane q of the row), fused multiply-adds in increasing q, each with
// the broadcast as its operand (5.7 cycles; a move and an fma take 10).  The leading
// wait is what a lane exchange needs after x is written, which the compiler does not
// see inside the block.  (Early clobber: acc is written before the last inputs are read,
// and an input of the same value could share its register otherwise; row_axpy8 alike.)
__device__ __forceinline__ double row_dot16(double acc, double x, const double (&t)[16])
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n\t"
        : "+&v"(acc)
        : "v"(x), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]),
          "v"(t[7]), "v"(t[8]), "v"(t[9]), "v"(t[10]), "v"(t[11]), "v"(t[12]), "v"(t[13]),
          "v"(t[14]), "v"(t[15]));
    return acc;
}
// r_q += f r_q(lane K of the row), q < 8
template <int K>
__device__ __forceinline__ void row_axpy8(double *r, double f)
{
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %0, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %1, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %2, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %3, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        : "+&v"(r[0]), "+&v"(r[1]), "+&v"(r[2]), "+&v"(r[3]), "+&v"(r[4]), "+&v"(r[5]),
          "+&v"(r[6]), "+&v"(r[7])
        : "v"(f), "n"(K));
}

// 1/a for the pivots of the eliminations: the hardware estimate refined by
// two Newton steps r <- r + r (1 - a r) (each squares the relative error),
// within an ulp of the rounded quotient for the normal, finite pivots of a
// positive definite elimination; five dependent operations instead of the
// ten of the correctly rounded division.
__device__ __forceinline__ double recip_nr(double a)
{
    double r = __builtin_amdgcn_rcp(a);
    double e = fma(-a, r, 1.0);
    r = fma(r, e, r);
    e = fma(-a, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float row_min(float x)
{
    x = fminf(x, dppf<kDppXor1>(x));
    x = fminf(x, dppf<kDppXor2>(x));
    x = fminf(x, dppf<kDppHalfMirror>(x));
    return fminf(x, dppf<kDppMirror>(x));
}
__device__ __forceinline__ double row_sum(double x)
{
    x += dppd<kDppXor1>(x);
    x += dppd<kDppXor2>(x);
    x += dppd<kDppHalfMirror>(x);
    return x + dppd<kDppMirror>(x);
}
// minimum over the four rows of a value that is uniform within each row
__device__ __forceinline__ float rows_min(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fminf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
__device__ __forceinline__ float wave_min(float x) { return rows_min(row_min(x)); }
// sum over the 64 lanes (every lane gets it): the row sums, then the row swaps
__device__ __forceinline__ double wave_sum(double x)
{
    x = row_sum(x);
    auto swap_add = [&](auto swap) {
        const uint64_t u = (uint64_t)__double_as_longlong(x);
        const auto lo = swap((uint32_t)u), hi = swap((uint32_t)(u >> 32));
        const double a = __longlong_as_double((long long)((uint64_t)lo[0] | ((uint64_t)hi[0] << 32)));
        const double b = __longlong_as_double((long long)((uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
        x = a + b;
    };
    swap_add([](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
    swap_add([](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
    return x;
}

// C(m, k), the size of a closed candidate set of m free dots with k raised (a
// table: the 64-bit divisions of the product form had cost the closed scorers
// some hundred instructions per pixel)
static __constant__ const uint16_t kBinomial[17][17] = {
    {1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 2, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 3, 3, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 4, 6, 4, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 5, 10, 10, 5, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 6, 15, 20, 15, 6, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 7, 21, 35, 35, 21, 7, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 8, 28, 56, 70, 56, 28, 8, 1, 0, 0, 0, 0, 0, 0, 0, 0},
    {1, 9, 36, 84, 126, 126, 84, 36, 9, 1, 0, 0, 0, 0, 0, 0, 0},
    {1, 10, 45, 120, 210, 252, 210, 120, 45, 10, 1, 0, 0, 0, 0, 0, 0},
    {1, 11, 55, 165, 330, 462, 462, 330, 165, 55, 11, 1, 0, 0, 0, 0, 0},
    {1, 12, 66, 220, 495, 792, 924, 792, 495, 220, 66, 12, 1, 0, 0, 0, 0},
    {1, 13, 78, 286, 715, 1287, 1716, 1716, 1287, 715, 286, 78, 13, 1, 0, 0, 0},
    {1, 14, 91, 364, 1001, 2002, 3003, 3432, 3003, 2002, 1001, 364, 91, 14, 1, 0, 0},
    {1, 15, 105, 455, 1365, 3003, 5005, 6435, 6435, 5005, 3003, 1365, 455, 105, 15, 1, 0},
    {1, 16, 120, 560, 1820, 4368, 8008, 11440, 12870, 11440, 8008, 4368, 1820, 560, 120, 16, 1},
};
__device__ __forceinline__ int64_t closed_states(int m, int k)
{
    return (k >= 0 && k <= m) ? kBinomial[m][k] : 0;
}

struct alignas(16) DiagRec {
    // inputs (written by the host, or by k_prep_batch): everything up to Cgd
    int32_t n, g, closed, nhat;
    double kT, t;
    int32_t prec, pad0;
    double Cdd[kMaxDot * kMaxDot];
    double Cgd[kMaxDot * kMaxGate];
    // computed by the prologue
    double one_c;                 // 1^T C_dd 1
    double c[kMaxDot];            // C_dd 1
    double A[kMaxDot * kMaxDot];  // C_dd^{-1}
    // matrix-core tables (dense box, n >= 9): low part = dots 0..7,
    // high part = dots 8..n-1; see qa_mfma.hip
    float T1[16][8];              // A_LH b_hi for the 4 row bits of the high index
    float T2[16][8];              // A_LH b_hi for the next 4 bits of the high index
    float Hhi[256];               // 1/2 b_hi^T A_HH b_hi
    float hlo[256];               // 1/2 b_lo^T A_LL b_lo
    float sumabs;                 // sum |A_ij| / 2, bound used by the error band
    float pad1[3];
    double hs[256];               // n <= 8: 1/2 s^T A s for every s in {0,1}^n
    // FP64 copies of the matrix-core tables (the near-tie re-score)
    double T1d[16][8], T2d[16][8];
    double Hhid[256], hlod[256];
    // bound-ordered search on the matrix cores (N >= 13): with S = (C_dd,HH)^{-1}, the Schur
    // complement of the low block in A, Hs = 1/2 b_hi^T S b_hi (1e30 past
    // 2^(N-8))
    float Hs[256];
    float sabsS;                  // sum |S_ij| / 2
    float pad2[3];
};

// Tables of the FP64 row kernels (qa_rows.hip), one per diagram (N >= 9): the
// low part is dots 0..5 (index lane, 64 values), the high part dots 6..N-1
// (index c = c6 + 64 k, c6 over dots 6..11).  Written by the setup; the part up
// to hs is copied to LDS as it is.
struct alignas(16) RowTab {
    double T[64][64];   // [c6][lane]: b_lo^T A_LH b_hi over dots 6..11
    double lo[4][64];   // sum of A_i,12+j over the lane's dots among 0..5
    double hi[4][64];   // the same over the lane's dots among 6..11
    float hs[16][64];   // 1/2 b_hi^T S b_hi, S = C_dd^{-1} over the high dots
    double hlo[64];     // 1/2 b^T A b over dots 0..5
    double hhi[64];     // the same over dots 6..11
    double hk[16];      // the same over dots 12..15
    float wB[10];       // closed arrays: w and 1 / (2 gamma) of the low-sum term
    float inv2g;
    float sabsS;        // sum |S_ij| / 2
};
constexpr size_t kRowTabLdsBytes = offsetof(RowTab, hlo);

// bytes of a DiagRec the host uploads (the inputs)
constexpr size_t kDiagInputBytes = offsetof(DiagRec, one_c);

struct alignas(64) PixRec {  // 256 bytes, two 128-byte lines
    double g0[kMaxDot];   // A (n0 - x_u)
    union {
        double u0;        // U(n0): setups without a bound (BoundSplit), for the softargmin
                          // and the scorers of every energy
        struct {          // setups with one, for the searches in bound order
            float eg;     // U(n0 + guess) - U(n0), from FP64; the guess is a state of the
                          // candidate set: the free dots whose x* rounds up, then the best
                          // single flip of a free dot if it lowers the energy (closed: the
                          // k free dots with the largest fractional parts)
            float slack;  // margin of the row kernels' bound test (see the setup)
        };
    };
    int32_t n0[kMaxDot];  // base state of the candidate set
    uint32_t free;        // dots that take both roundings
    int32_t k;            // closed: number of raised free dots; -1 open
    // lower bound of the states of a high part b_hi (N >= 9):
    // K + b_hi^T s + 1/2 b_hi^T S b_hi, s = S (n0 - x_u)_hi; the high part is
    // dots 8..N-1 or 6..N-1, as the setup was asked for (BoundSplit)
    float s[10];
    float K;
    float mu;             // closed: -1^T A_LL^{-1} g_lo (the low sum of the free minimiser)
};
static_assert(sizeof(PixRec) == 256, "two lines");

struct alignas(8) SavedRec {
    double emin;          // reference energy (N <= 8: the smallest candidate energy)
    double Z;             // sum exp(-(E - emin)/kT)
    double nb[kMaxDot];   // <n> - n0 = sum_s pi_s 1_s (zero beyond n)
    int32_t n0[kMaxDot];
    uint32_t free;
    int32_t k;
};

// one diagram of a ragged batch, as uploaded by the host (work order)
struct alignas(8) BatchHdr {
    int32_t n, g, closed, nhat;
    double kT, t;
    int64_t v_off;    // element offset of the diagram's P x G voltages
    int64_t out_off;  // element offset of its P x N outputs
    int64_t P;        // pixels
    int64_t mat_off;  // offset of C_dd (n x n) then C_gd (n x g) in the matrix buffer
    int64_t tile0;    // first 64-pixel work item of the diagram
    // swept diagrams (nx > 0): the voltages are formed from the sweep at
    // grid_off in the matrix buffer: v0, e1, e2 (g each), then a0, da, a1,
    // b0, db, b1 (see VGrid); P = nx * ny
    int64_t grid_off;
    int32_t nx, ny;
};

// An affine sweep of the gate voltages over a raster of nx x ny pixels,
// pixel p = j nx + i:  V(i, j) = (v0 + a_i e1) + b_j e2 with a_i = i da + a0
// (the last a_i is a1 itself) and b_j alike.  These are the values that
// numpy's linspace and broadcast arithmetic give, rounded the same way (no
// fused multiply-add), so a sweep and the explicit voltages it describes
// give bitwise identical results.  on = 0: explicit voltages instead.
struct VGrid {
    double v0[kMaxGate], e1[kMaxGate], e2[kMaxGate];
    double a0, da, a1, b0, db, b1;
    int64_t nx, ny;
    int32_t on, pad;
};

// point i of num equally spaced points from start to stop (step = (stop -
// start) / (num - 1), 0 for one point), as numpy's linspace forms it
// (contraction into fused multiply-adds is off in both: each product and
// sum is rounded on its own)
__device__ __forceinline__ double lin_point(int32_t i, int32_t num, double start, double step,
                                            double stop)
{
#pragma clang fp contract(off)
    const double t = (double)i * step;
    return (num > 1 && i == num - 1) ? stop : t + start;
}
// v0_k + a e1_k + b e2_k, each operation rounded on its own
__device__ __forceinline__ double sweep_volt(double v0, double e1, double e2, double a, double b)
{
#pragma clang fp contract(off)
    const double s = v0 + a * e1;
    return s + b * e2;
}
// the sweep coordinates (a, b) of pixel p (Grid: VGrid, SetupIn)
template <typename Grid>
__device__ __forceinline__ void grid_ab(const Grid &G, int64_t p, double &a, double &b)
{
    // (a sweep has fewer than 2^31 pixels)
    const uint32_t nx = (uint32_t)G.nx, row = (uint32_t)p / nx;
    a = lin_point((int32_t)((uint32_t)p - row * nx), (int32_t)nx, G.a0, G.da, G.a1);
    b = lin_point((int32_t)row, (int32_t)G.ny, G.b0, G.db, G.b1);
}
// gate k's voltage at sweep coordinates (a, b)
__device__ __forceinline__ double grid_v(const VGrid &G, int k, double a, double b)
{
    return sweep_volt(G.v0[k], G.e1[k], G.e2[k], a, b);
}

// The inputs of a DiagRec carried in a kernel's arguments (no host staging
// buffer and no copy call): part 0 writes the header and C_dd, part 1 rows
// [row0, row1) of C_gd; entries past the problem's n x n and n x g are
// written as zeros, so the record's padding is the same whatever an earlier
// call left there.  A chunk holds at most kChunkDoubles matrix entries.
constexpr int kChunkDoubles = 256;
struct InputChunk {
    int32_t n, g, closed, nhat;
    double kT, t;
    int32_t prec;
    int32_t part;        // 0: header and C_dd; 1: C_gd rows [row0, row1)
    int32_t row0, row1;  // part 1: rows of the padded C_gd written by this chunk
    double v[kChunkDoubles];  // part 0: C_dd, n x n; part 1: rows row0.. of C_gd, each g long
};

// A call's inputs as arguments of the setup kernel: v holds the lower triangle of
// C_dd by rows, C_gd (n x g) and, for a sweep, v0, e1, e2 (g each).  Against a copy
// into the record ahead of the kernel (with the event that guards its pinned
// source) a call takes 4.4 us for 9.3 at the host and a launch less on the GPU; 256
// or 640 blocks that read 3 KB of arguments take no longer than from memory.  440
// doubles keep the kernel's arguments below 4 KB: 16 dots with 16 gates and a sweep.
constexpr int kSetupInDoubles = 440;
struct SetupIn {
    int32_t n, g, closed, nhat;
    double kT, t;
    int32_t prec, on;  // on: a sweep, of
    double a0, da, a1, b0, db, b1;
    int64_t nx, ny;
    double v[kSetupInDoubles];
};

// which lower bound of a high part the setup forms per pixel (N >= 9): none,
// with eight low dots (the matrix-core scorer) or with six (the FP64 row
// kernels)
enum BoundSplit : int { kBoundNone = 0, kBoundLow6 = 6, kBoundLow8 = 8 };

// the setup kernel: one wave for the prologue, seven for the pixels
constexpr int kSetupPixThreads = 7 * kWave;
// its grid is largest for 16-lane pixel groups
constexpr int64_t setup_blocks_max(int64_t P)
{
    return P < 1 ? 1 : (P * kMaxDot + kSetupPixThreads - 1) / kSetupPixThreads;
}

// -------------------------------------------------------------------------
// launch wrappers (qa_kernels.hip); all enqueue on `s` and return the HIP
// error of the launch.
// -------------------------------------------------------------------------
hipError_t launch_zero_i64(int64_t *p, int n, hipStream_t s);
// one chunk of a diagram's inputs into dr
hipError_t launch_put_inputs(DiagRec *dr, const InputChunk &c, hipStream_t s);
// prologue of a diagram whose setup has not run (the adjoint by itself); also zeroes the
// nzero doubles at zero when given
hipError_t launch_prep(DiagRec *dr, hipStream_t s, double *zero = nullptr, int64_t nzero = 0);
// prologue (every block; block 0 also stores A and the tables into dr and
// clears the kCounterWords counters) and setup of every pixel; the per-block
// counts {pixels, QP, doubled, QP failures, gaps below 1e-9, candidates} go to
// bstats[kBstatWords * block] for
// setup_blocks(P, n_dot) blocks; split: the bound terms the scorer of this call
// reads (kBoundNone for N <= 8); rt: receives the row tables (N >= 9, needed for
// kBoundLow6) or NULL; x_out (P x N) / flags_out (P) are optional
// copies of x*; grid, when given and on, replaces the voltages V; in: the inputs
// (with the sweep) as arguments, stored into dr by the kernel, or NULL when dr
// holds them; n_out (N <= 8): the kernel scores too and writes the ground states
// there instead of the pixel records and dr's tables.  P >= 1.
constexpr int kBstatWords = 6;
int64_t setup_blocks(int64_t P, int n_dot);
hipError_t launch_setup(DiagRec *dr, const double *V, int64_t P, PixRec *pr, int64_t *counters,
                        int32_t *bstats, int n_dot, bool closed, BoundSplit split, RowTab *rt,
                        hipStream_t s, double *x_out = nullptr, int32_t *flags_out = nullptr,
                        const VGrid *grid = nullptr,
                        const SetupIn *in = nullptr, int32_t *n_out = nullptr);
// T = 0 argmin in FP64 over the candidate set of every pixel, every energy (N >= 9)
hipError_t launch_score_fp64(const DiagRec *dr, const PixRec *pr, int64_t P, int32_t *n_out,
                             int64_t *counters, int n_dot, hipStream_t s);
// the same for N >= 9 in bound order (qa_rows.hip; setup split kBoundLow6);
// mode as for launch_score_mfma
hipError_t launch_rows_gs(const RowTab *rt, const PixRec *pr, int64_t P, int mode, int32_t *n_out,
                          int64_t *counters, int n_dot, hipStream_t s);
// matrix-core scorer at T = 0; mode 0: the dense box, 1: the sub-box of each
// pixel's free dots (thresholded), 2: closed arrays (subsets of the free
// dots with k raised); near ties re-scored in FP64 inside the kernel.  Every
// state of the set, or (exhaustive false: modes 0 and 1, N >= 13, split BF16, setup
// split kBoundLow8) searched in bound order.
hipError_t launch_score_mfma(const DiagRec *dr, const PixRec *pr, int64_t P, int prec, int mode,
                             bool exhaustive, int32_t *n_out, int64_t *counters, int n_dot,
                             hipStream_t s);
// softargmin of N >= 9 dots as FP64 matrix products (qa_soft.hip), for couplings
// and temperatures that soft_mm_range (qa_api.hip) admits
hipError_t launch_soft_mm(const DiagRec *dr, const RowTab *rt, const PixRec *pr, int64_t P,
                          double *nbar, SavedRec *saved, int n_dot, bool closed, hipStream_t s);
// its adjoint (9 <= N <= 12), into the same accumulators as launch_soft_bwd
hipError_t launch_soft_mm_bwd(const DiagRec *dr, const RowTab *rt, const double *V, int64_t P,
                              const double *gbar, const SavedRec *saved, double *acc,
                              double *gradV, int n_dot, bool closed, hipStream_t s,
                              const VGrid *grid = nullptr);
// the row tables (without the bound's) of a record whose prologue has run
hipError_t launch_row_tab(const DiagRec *dr, RowTab *rt, hipStream_t s);
// softargmin: the table form (N <= 8), or a walk over every candidate
hipError_t launch_soft_fwd(const DiagRec *dr, const PixRec *pr, int64_t P, double *nbar,
                           SavedRec *saved, int64_t *counters, int n_dot, hipStream_t s);
// adjoint partial sums: kBwdReplicas copies of (dL/dA, kMaxDot^2; dL/dC_gd,
// kMaxDot x kMaxGate), block b adding into copy b mod kBwdReplicas, so that
// fewer blocks contend for one address; zero on entry, and left zero by the
// final kernel, which adds the copies up
constexpr int kBwdReplicas = 8;
constexpr int kBwdAccWords = kMaxDot * kMaxDot + kMaxDot * kMaxGate;
hipError_t launch_soft_bwd(const DiagRec *dr, const double *V, int64_t P,
                           const double *gbar, const SavedRec *saved, double *acc,
                           double *gradV, int n_dot, hipStream_t s, const VGrid *grid = nullptr);
hipError_t launch_soft_bwd_final(const DiagRec *dr, double *acc, double *grad_cdd,
                                 double *grad_cgd, hipStream_t s);
// charge-sensor response (qa_sensor.hip): the last n_sensor dots of the problem in
// `in` (or in dr when NULL) are sensors; array charges from n_int or n_dbl
// (P x (n - n_sensor)); noise draws optional (NULL: none); parity: scratch of
// kSensorParities words; signal P x n_sensor
constexpr int kSensorParities = 1024;
hipError_t launch_sensor(const DiagRec *dr, const SetupIn *in, int n_dot, int n_sensor, int shape,
                         double gamma, const double *V, int64_t P, const int32_t *n_int,
                         const double *n_dbl, const double *white_draws, double white,
                         const double *pink_draws, double pink, int octaves,
                         const double *jump_draws, double jump, double rate, int32_t *parity,
                         double *signal, hipStream_t s);
// ragged batch (qa_batch.hip): prologue of every diagram, then one
// kernel over all 64-pixel work items
hipError_t launch_prep_batch(const BatchHdr *hdr, const double *mats, DiagRec *recs, int n_diag,
                             int32_t *owner, int64_t *counters, hipStream_t s);
hipError_t launch_batch(const BatchHdr *hdr, const DiagRec *recs, const double *mats,
                        const int32_t *owner, int64_t tiles, const double *V, int32_t *n_out,
                        double *nbar, int64_t *counters, int max_dot, hipStream_t s);

}  // namespace qa
