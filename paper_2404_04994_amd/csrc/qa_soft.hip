// qa_soft.hip -- softargmin (Sec. 4.2, Eq. softargmin) of 9 <= N <= 16 dots as FP64
// matrix products.
//
// With the dots split into a low part (dots 0..5, 64 states l), a middle part
// (dots 6..11, 64 states c) and a high part (dots 12..N-1, states k), a
// candidate's energy relative to U(n0) is
//     E(l, c, k) = a_k(l) + c_k(c) + T(c, l),   T = b_l^T A b_c,
// so its weight is a product of three factors, exp(-E/kT) = F1_k(l) F2_k(c) W(c, l),
// and W depends on the diagram alone.  All sums over the 4096 states of one
// (pixel, k) are then
//     sum_l [..] F1(l) Y(l),   Y(l) = sum_c W(c, l) F2(c),
//     sum_c [..] F2(c) X(c),   X(c) = sum_l W(c, l) F1(l),
// two products of the same 64 x 64 matrix with a column per (pixel, k): 16
// columns at a time, v_mfma_f64_16x16x4_f64, W in registers for the whole kernel
// (each of a block's four waves keeps 16 rows of W and of W^T).  That is 4
// flops per candidate and 128 exponentials per 4096 candidates; walking the
// candidates took an exponential and some forty FP64 operations each.
//
// Range: T is taken around the middle of the box, T' = (b_l - 1/2)^T A (b_c - 1/2)
// (the linear rest goes to a and c), and a and c from their smallest values, so
// that F1, F2 <= 1 and |log W| <= max|T'| / kT.  A candidate within exp(-52) of
// the largest weight then has every factor above exp(-2 max|T'| / kT - 52): for
// max|T'| <= 300 kT nothing that counts is lost (the host checks it; smaller kT
// walks the candidates).
//
// Closed arrays: a low state of popcount m pairs with the middle states of
// popcount K - m only (K = k - popc of the high state).  The middle states are
// ordered by popcount, a matrix step never crosses a class (19 steps of four
// instead of 16), each class keeps its own accumulator, and the sums pick the
// one class of each low state; the other product alike.  F1 and F2 are then
// taken from the smallest values of their class, and a pair of classes has its
// own factor, so the same range holds within each.
//
// Bound: for 16 dots the vector instructions around the products (some 600 per
// wave and set of columns beside 32 products of 64 cycles) at two waves per SIMD,
// which is what the registers allow; launch and prologue latency for few
// pixels.  Measured against the walk over the candidates (one wave per pixel):
// 16 dots, 10^4 pixels 10900 -> 110 us; 12 dots, 4096 pixels 400 -> 9.7 us; error
// against 64 bits 3.3e-15 -> 1.8e-15 (16 dots, kT = 0.01).
#include "qa_device.h"

namespace qa {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

constexpr int kSoftThreads = 256;
constexpr int kSoftRows = 16;  // (pixel, k) columns per batch

// states ordered by popcount, each class padded to a multiple of four slots
constexpr int kClassStep[8] = {0, 1, 3, 7, 12, 16, 18, 19};  // first step of class m
struct ClassOrder {
    uint8_t slot[64];   // slot of a state
    uint8_t state[76];  // state of a slot (64: padding)
};
constexpr ClassOrder class_order()
{
    ClassOrder o{};
    int fill[7] = {};
    for (int s = 0; s < 76; ++s) o.state[s] = 64;
    for (int s = 0; s < 64; ++s) {
        const int m = __builtin_popcount(s);
        o.slot[s] = (uint8_t)(4 * kClassStep[m] + fill[m]++);
        o.state[o.slot[s]] = (uint8_t)s;
    }
    return o;
}
static __constant__ const ClassOrder kOrder = class_order();

// exp(x) for -1100 <= x <= 700 (zero at the lower end): x = n ln 2 + r, |r| <= ln 2 / 2, and a
// polynomial of degree 11 for exp(r), the interpolant of (exp(r) - 1 - r) / r^2 at
// Chebyshev nodes (relative error 2e-17 before rounding).
__device__ __forceinline__ double exp_small(double x)
{
    const double n = rint(x * 0x1.71547652b82fep+0);
    double r = fma(n, -0x1.62e42fefa39efp-1, x);
    r = fma(n, -0x1.abc9e3b39803fp-56, r);
    double p = 0x1.af390e40bdeadp-26;
    p = fma(p, r, 0x1.2891a8fe8d7d2p-22);
    p = fma(p, r, 0x1.71de0d81d74e1p-19);
    p = fma(p, r, 0x1.a019b8ef350abp-16);
    p = fma(p, r, 0x1.a01a01a7d093cp-13);
    p = fma(p, r, 0x1.6c16c17893938p-10);
    p = fma(p, r, 0x1.11111111109a0p-7);
    p = fma(p, r, 0x1.5555555553d4fp-5);
    p = fma(p, r, 0x1.5555555555556p-3);
    p = fma(p, r, 0x1.0000000000001p-1);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)n);
}

// exp(x) for x <= 0, zero below -1100
__device__ __forceinline__ double exp_neg(double x) { return exp_small(fmax(x, -1100.0)); }

// value of the lane in the neighbouring 16-lane row (rows 0-1, 2-3) or half
__device__ __forceinline__ double other_row(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const int odd = threadIdx.x >> 4 & 1;
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)(odd ? lo[0] : lo[1]) |
                                            ((uint64_t)(odd ? hi[0] : hi[1]) << 32)));
}
__device__ __forceinline__ double other_half(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const int odd = threadIdx.x >> 5 & 1;
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)(odd ? lo[0] : lo[1]) |
                                            ((uint64_t)(odd ? hi[0] : hi[1]) << 32)));
}
// minimum over a 16-lane row
__device__ __forceinline__ double row_min_d(double x)
{
    x = fmin(x, dppd<kDppXor1>(x));
    x = fmin(x, dppd<kDppXor2>(x));
    x = fmin(x, dppd<kDppHalfMirror>(x));
    return fmin(x, dppd<kDppMirror>(x));
}

// slot of a state in the order of a product's columns
template <bool CLOSED>
__device__ __forceinline__ int soft_slot(int s)
{
    return CLOSED ? (int)kOrder.slot[s] : s;
}

constexpr double kNoState = 0x1p1000;  // energy of a state outside the candidate set

// The matrix operand of one wave: rows 16 w .. 16 w + 15 of W^T (low states, over
// the middle states) and of W, lane (m, q) holding row m, column of slot 4 t + q.
template <int STEPS>
struct SoftW {
    double y[STEPS], x[STEPS];
};
// T: the diagram's table in LDS, columns of kTStride doubles
constexpr int kTStride = 65;
template <bool CLOSED, int STEPS>
__device__ __forceinline__ void soft_w(const double *T, double ikT, int w, SoftW<STEPS> &o)
{
    const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
    const int row = 16 * w + m;
    const double tl = T[63 * kTStride + row], tc = T[row * kTStride + 63];
    const double tt = 0.25 * T[63 * kTStride + 63];
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        const int s = CLOSED ? (int)kOrder.state[4 * t + q] : 4 * t + q;
        const int sc = s & 63;
        // T' of (middle s, low row) and of (middle row, low s), of either sign (below
        // 300 kT by the host's check); padding slots are zero
        const double ey = (T[sc * kTStride + row] - 0.5 * (tl + T[sc * kTStride + 63])) + tt;
        const double ex = (T[row * kTStride + sc] - 0.5 * (tc + T[63 * kTStride + sc])) + tt;
        const double wy = exp_small(-ey * ikT), wx = exp_small(-ex * ikT);
        o.y[t] = s < 64 ? wy : 0.0;
        o.x[t] = s < 64 ? wx : 0.0;
        // finished here: the compiler sinks the last steps of every exponential
        // past the barrier otherwise, and keeps twice the registers until then
        asm volatile("" : "+v"(o.y[t]), "+v"(o.x[t])::"memory");
    }
}

// acc[m] += rows of W times the columns F (LDS, stride doubles per column)
template <bool CLOSED, int STEPS, int CLASSES>
__device__ __forceinline__ void soft_product(const double (&w)[STEPS], const double *F, int stride,
                                             f64x4_t (&acc)[CLASSES])
{
    const int lane = threadIdx.x & 63;
    const double *col = F + (lane & 15) * stride + (lane >> 4);
    static_for_dev<0, STEPS>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int m = CLOSED ? (t < 1 ? 0 : t < 3 ? 1 : t < 7 ? 2 : t < 12 ? 3 : t < 16 ? 4 : t < 18 ? 5 : 6) : 0;
        acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[t], col[4 * t], acc[m], 0, 0, 0);
    });
}

// element i of a lane's tile, state s = 16 w + q + 4 i: of the accumulators of a
// closed product the one of the partner's popcount K - popc(s)
template <bool CLOSED, int CLASSES>
__device__ __forceinline__ double soft_pick(const f64x4_t (&acc)[CLASSES], int i, int s, int K)
{
    double y = acc[0][i];
    if (CLOSED) {
        const int want = K - __popc((uint32_t)s);
        y = want == 0 ? y : 0.0;
#pragma unroll
        for (int m = 1; m < CLASSES; ++m) y = want == m ? acc[m][i] : y;
    }
    return y;
}

// The five sums of a column over the tile's 16 states: all of them and those with
// bit 0..3 of s set, from the lane's four elements v; every lane of the column
// ends with them.
__device__ __forceinline__ void soft_sums5(const double (&v)[4], double (&out)[5])
{
    const int q = (threadIdx.x & 63) >> 4;
    double t = (v[0] + v[1]) + (v[2] + v[3]);
    double b2 = v[1] + v[3], b3 = v[2] + v[3];
    const double to = other_row(t);
    double b0 = (q & 1) ? t : to;
    t += to;
    b2 += other_row(b2);
    b3 += other_row(b3);
    const double th = other_half(t);
    const double b1 = (q & 2) ? t : th;
    out[0] = t + th;
    out[1] = b0 + other_half(b0);
    out[2] = b1;
    out[3] = b2 + other_half(b2);
    out[4] = b3 + other_half(b3);
}
// sum of dot 0..5 of a product's part sums (part[wave][..][column])
template <typename Part>
__device__ __forceinline__ double soft_dot_sum(const Part &part, int prod, int dot, int col)
{
    if (dot < 4)
        return (part[0][prod][1 + dot][col] + part[1][prod][1 + dot][col]) +
               (part[2][prod][1 + dot][col] + part[3][prod][1 + dot][col]);
    return part[dot == 4 ? 1 : 2][prod][0][col] + part[3][prod][0][col];
}

template <bool CLOSED>
struct SoftLds {
    static constexpr int kSteps = CLOSED ? 19 : 16;
    static constexpr int kStride = 4 * kSteps + 2;  // columns two doubles apart in the banks
    double F1[kSoftRows][kStride], F2[kSoftRows][kStride];
    double part[4][2][5][kSoftRows];  // [wave][product][sum][column]
    // closed: smallest energies of each class (low, middle) as ordered integers
    unsigned long long cmin[CLOSED ? 2 : 1][kSoftRows][8];
    double ref[kSoftRows];            // smallest a + c of the column
    PixRec rec[2][kSoftRows];
};

// The factors of a batch's columns: thread (column = tid / 16, s = tid mod 16 + 16 i)
// forms F1 and F2 of four states each and the column's reference.
struct SoftConst {
    double a[4], c[4];  // quadratic terms of the thread's states for the column's k
    double kbit[4];     // bits of k
    double bit[4];      // bits 0..3 of the thread's states
};
template <int NK>
__device__ __forceinline__ void soft_const(const RowTab *__restrict__ rt, const double *T,
                                           SoftConst &o)
{
    const int s0 = threadIdx.x & 15, k = (threadIdx.x >> 4) & ((1 << NK) - 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        o.kbit[j] = (k >> j & 1) ? 1.0 : 0.0;
        o.bit[j] = (s0 >> j & 1) ? 1.0 : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int s = s0 + 16 * i;
        double a = rt->hlo[s] + 0.5 * T[63 * kTStride + s];
        double c = (rt->hhi[s] + 0.5 * T[s * kTStride + 63]) - 0.25 * T[63 * kTStride + 63] + rt->hk[k];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a = fma(o.kbit[j], rt->lo[j][s], a);
            c = fma(o.kbit[j], rt->hi[j][s], c);
        }
        o.a[i] = a;
        o.c[i] = c;
    }
}

// doubles as integers of the same order (energies that are not numbers, all of a pixel's
// then, come out as classes without a smallest energy: no weights, charges 0 / 0)
__device__ __forceinline__ unsigned long long ordered(double x)
{
    const long long u = __double_as_longlong(x);
    return (unsigned long long)u ^ ((unsigned long long)(u >> 63) | (1ull << 63));
}
__device__ __forceinline__ double from_ordered(unsigned long long o)
{
    return __longlong_as_double((long long)(o ^ (~((long long)o >> 63) | (1ll << 63))));
}

// f1 and f2 of the thread's four states for the pixel (g0, free dots, raised
// count K_all); returns the column's reference.  The factor of a pair of classes
// goes into f1.  (Contains a block barrier when CLOSED.)
template <bool CLOSED, int NK, typename Lds>
__device__ __forceinline__ double soft_factors(const double *g0, uint32_t fm, int K_all,
                                               const SoftConst &o, double ikT, Lds &L,
                                               double (&f1)[4], double (&f2)[4])
{
    const int s0 = threadIdx.x & 15, colm = threadIdx.x >> 4;
    const int kk = colm & ((1 << NK) - 1);
    double gl = 0.0, gm = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        gl = fma(o.bit[j], g0[j], gl);
        gm = fma(o.bit[j], g0[6 + j], gm);
    }
#pragma unroll
    for (int j = 0; j < NK; ++j) gm = fma(o.kbit[j], g0[12 + j], gm);
    const bool khi = ((uint32_t)kk & ~(fm >> 12)) == 0;  // raises no fixed dot of 12..15
    double e1[4], e2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t s = (uint32_t)(s0 + 16 * i);
        const double g45 = (i & 1 ? g0[4] : 0.0) + (i & 2 ? g0[5] : 0.0);
        const double h45 = (i & 1 ? g0[10] : 0.0) + (i & 2 ? g0[11] : 0.0);
        e1[i] = (s & ~fm & 63u) ? kNoState : (o.a[i] + gl) + g45;
        e2[i] = (s & ~(fm >> 6) & 63u) || !khi ? kNoState : (o.c[i] + gm) + h45;
    }
    if constexpr (!CLOSED) {
        const double r1 = row_min_d(fmin(fmin(e1[0], e1[1]), fmin(e1[2], e1[3])));
        const double r2 = row_min_d(fmin(fmin(e2[0], e2[1]), fmin(e2[2], e2[3])));
        const double rf = r2 < kNoState ? r2 : 0.0;  // (none of the column's states: all zero)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f1[i] = exp_neg((r1 - e1[i]) * ikT);
            f2[i] = exp_neg((rf - e2[i]) * ikT);
            if (i & 1) __builtin_amdgcn_sched_barrier(0);
        }
        return r1 + r2;
    } else {
        // states s0 + 16 i have popcounts pl, pl + 1, pl + 1, pl + 2
        const int pl = __popc((uint32_t)s0);
        atomicMin(&L.cmin[0][colm][pl], ordered(e1[0]));
        atomicMin(&L.cmin[0][colm][pl + 1], ordered(fmin(e1[1], e1[2])));
        atomicMin(&L.cmin[0][colm][pl + 2], ordered(e1[3]));
        atomicMin(&L.cmin[1][colm][pl], ordered(e2[0]));
        atomicMin(&L.cmin[1][colm][pl + 1], ordered(fmin(e2[1], e2[2])));
        atomicMin(&L.cmin[1][colm][pl + 2], ordered(e2[3]));
        __syncthreads();
        // lane m: low class m pairs with middle class K - m
        const int a = K_all - __popc((uint32_t)kk) - s0;
        double rr = kNoState;
        if (s0 < 7 && a >= 0 && a < 7) {
            const double r1 = from_ordered(L.cmin[0][colm][s0]), r2 = from_ordered(L.cmin[1][colm][a]);
            rr = r1 < kNoState && r2 < kNoState ? r1 + r2 : kNoState;
        }
        const double ref = row_min_d(rr);
        const double pair = rr < kNoState ? exp_neg((ref - rr) * ikT) : 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = pl + (i == 0 ? 0 : (i == 3 ? 2 : 1));
            const double r1 = from_ordered(L.cmin[0][colm][m]), r2 = from_ordered(L.cmin[1][colm][m]);
            const double c = __shfl(pair, m, 16);
            f1[i] = e1[i] < kNoState ? exp_neg((r1 - e1[i]) * ikT) * c : 0.0;
            f2[i] = e2[i] < kNoState ? exp_neg((r2 - e2[i]) * ikT) : 0.0;
            if (i & 1) __builtin_amdgcn_sched_barrier(0);
        }
        return ref;
    }
}

// Block b takes batches b, b + gridDim.x, ...: 16 >> NK pixels of 2^NK high
// states, NK = max(0, N - 12).
template <bool CLOSED, int NK>
__global__ __launch_bounds__(kSoftThreads, 2) void k_soft_mm(const DiagRec *__restrict__ dr,
                                                             const RowTab *__restrict__ rt,
                                                             const PixRec *__restrict__ pr, int64_t P,
                                                             double *__restrict__ nbar,
                                                             SavedRec *__restrict__ saved, int n)
{
    constexpr int STEPS = SoftLds<CLOSED>::kSteps, STRIDE = SoftLds<CLOSED>::kStride;
    constexpr int CLASSES = CLOSED ? 7 : 1;
    // the table T during the prologue, then the batch's buffers
    __shared__ union Shared {
        double T[64 * kTStride];
        SoftLds<CLOSED> L;
        __device__ Shared() {}
    } sh;
    SoftLds<CLOSED> &L = sh.L;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int per = kSoftRows >> NK;  // pixels per batch
    const int64_t batches = (P + per - 1) / per;
    const double ikT = 1.0 / dr->kT;
    for (int r = 0; r < 16; ++r) {
        const int e = r * kSoftThreads + tid;
        sh.T[(e >> 6) * kTStride + (e & 63)] = (&rt->T[0][0])[e];
    }
    // record dwords 4 (tid mod 16) .. + 3 of the batch's pixel tid / 16
    auto fetch = [&](int64_t b) -> uint4 {
        int64_t p = b * per + (tid >> 4);
        p = p < P ? p : P - 1;
        return (tid >> 4) < per ? reinterpret_cast<const uint4 *>(pr + p)[tid & 15] : uint4{};
    };
    uint4 next = fetch(blockIdx.x);
    __syncthreads();
    SoftW<STEPS> W;
    soft_w<CLOSED, STEPS>(sh.T, ikT, w, W);
    SoftConst sc;
    soft_const<NK>(rt, sh.T, sc);
    __syncthreads();
    for (int i = tid; i < kSoftRows * STRIDE; i += kSoftThreads) {
        (&L.F1[0][0])[i] = 0.0;  // the padding slots stay zero
        (&L.F2[0][0])[i] = 0.0;
    }
    int buf = 0;
    for (int64_t b = blockIdx.x; b < batches; b += gridDim.x, buf ^= 1) {
        if ((tid >> 4) < per) reinterpret_cast<uint4 *>(&L.rec[buf][tid >> 4])[tid & 15] = next;
        if (CLOSED) (&L.cmin[0][0][0])[tid] = ordered(kNoState);
        if (b + gridDim.x < batches) next = fetch(b + gridDim.x);
        __syncthreads();
        {
            const PixRec *r = &L.rec[buf][(tid >> 4) >> NK];
            double f1[4], f2[4];
            const double ref =
                soft_factors<CLOSED, NK>(r->g0, r->free, r->k, sc, ikT, L, f1, f2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = soft_slot<CLOSED>((tid & 15) + 16 * i);
                L.F1[tid >> 4][at] = f1[i];
                L.F2[tid >> 4][at] = f2[i];
            }
            if ((tid & 15) == 0) L.ref[tid >> 4] = ref;
        }
        __syncthreads();
        {
            const int col = tid & 15;
            const int K = CLOSED ? L.rec[buf][col >> NK].k - __popc((uint32_t)(col & ((1 << NK) - 1))) : 0;
            double v[4], sy[5], sx[5];
            auto times = [&](const double (*F)[STRIDE], const f64x4_t (&acc)[CLASSES]) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int s = 16 * w + ((tid & 63) >> 4) + 4 * i;
                    v[i] = F[col][soft_slot<CLOSED>(s)] * soft_pick<CLOSED>(acc, i, s, K);
                }
            };
            {
                f64x4_t y[CLASSES] = {};
                soft_product<CLOSED, STEPS, CLASSES>(W.y, &L.F2[0][0], STRIDE, y);
                times(L.F1, y);
                soft_sums5(v, sy);
            }
            {
                f64x4_t x[CLASSES] = {};
                soft_product<CLOSED, STEPS, CLASSES>(W.x, &L.F1[0][0], STRIDE, x);
                times(L.F2, x);
                soft_sums5(v, sx);
            }
            if ((tid & 63) < 16) {
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    L.part[w][0][j][col] = sy[j];
                    L.part[w][1][j][col] = sx[j];
                }
            }
        }
        __syncthreads();
        // thread (column, item): item 0 the normaliser, 1..6 dots 0..5, 7..12 dots
        // 6..11, 13..16 dots 12..15; the columns of a pixel are added up by the
        // lanes of its 2^nk columns
        const int col = tid & 15;
        const double ref = L.ref[col];
        auto over_k = [&](double v, auto &&op) {
            if constexpr (NK >= 1) v = op(v, dppd<kDppXor1>(v));
            if constexpr (NK >= 2) v = op(v, dppd<kDppXor2>(v));
            if constexpr (NK >= 3) v = op(v, dppd<kDppHalfMirror>(v));
            if constexpr (NK >= 4) v = op(v, dppd<kDppMirror>(v));
            return v;
        };
        const double low = over_k(ref, [](double u, double v) { return fmin(u, v); });
        const double scale = exp_neg((low - ref) * ikT);
        const double zc = scale * ((L.part[0][0][0][col] + L.part[1][0][0][col]) +
                                   (L.part[2][0][0][col] + L.part[3][0][0][col]));
        const double Z = over_k(zc, [](double u, double v) { return u + v; });
        const int64_t p = b * per + (col >> NK);
        const bool writer = (col & ((1 << NK) - 1)) == 0 && p < P;
        const PixRec *r = &L.rec[buf][col >> NK];
        for (int item = tid >> 4; item < 17; item += 16) {
            double v = 0.0;
            if (item >= 13) {
                v = (col >> (item - 13) & 1) && item - 13 < NK ? zc : 0.0;
            } else if (item >= 1) {
                v = scale * soft_dot_sum(L.part, item >= 7 ? 1 : 0, (item - 1) % 6, col);
            }
            v = over_k(v, [](double u, double t) { return u + t; });
            if (!writer) continue;
            if (item == 0) {
                if (saved) {
                    SavedRec *o = saved + p;
                    o->emin = r->u0 + low;
                    o->Z = Z;
                    o->free = r->free;
                    o->k = r->k;
                }
                continue;
            }
            const int d = item - 1;
            const double f = d < n ? v / Z : 0.0;
            if (d < n) nbar[p * n + d] = (double)r->n0[d] + f;
            if (saved) {
                saved[p].nb[d] = f;
                saved[p].n0[d] = r->n0[d];
            }
        }
    }
}

// blocks for a number of batches: at most as many as the chip keeps resident
// (cached per kernel and device)
template <typename Kernel>
static unsigned soft_blocks(Kernel kernel, int (&cache)[64], int64_t batches)
{
    int dev = 0;
    int64_t most = 512;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) {
        int cus = 0, per_cu = 0;
        if (!cache[dev] &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kSoftThreads, 0) == hipSuccess)
            cache[dev] = cus * per_cu;
        if (cache[dev] > 0) most = cache[dev];
    }
    return (unsigned)(batches < most ? batches : most);
}

hipError_t launch_soft_mm(const DiagRec *dr, const RowTab *rt, const PixRec *pr, int64_t P,
                          double *nbar, SavedRec *saved, int n_dot, bool closed, hipStream_t s)
{
    if (n_dot < 9 || n_dot > kMaxDot || !rt) return hipErrorInvalidValue;
    if (P <= 0) return hipSuccess;
    const int nk = n_dot > 12 ? n_dot - 12 : 0;
    const int64_t batches = (P + (kSoftRows >> nk) - 1) / (kSoftRows >> nk);
    static int cache[10][64];
    auto go = [&](auto kernel, int slot) {
        hipLaunchKernelGGL(kernel, dim3(soft_blocks(kernel, cache[slot], batches)),
                           dim3(kSoftThreads), 0, s, dr, rt, pr, P, nbar, saved, n_dot);
        return hipGetLastError();
    };
    switch (2 * nk + (closed ? 1 : 0)) {
    case 0: return go(k_soft_mm<false, 0>, 0);
    case 1: return go(k_soft_mm<true, 0>, 1);
    case 2: return go(k_soft_mm<false, 1>, 2);
    case 3: return go(k_soft_mm<true, 1>, 3);
    case 4: return go(k_soft_mm<false, 2>, 4);
    case 5: return go(k_soft_mm<true, 2>, 5);
    case 6: return go(k_soft_mm<false, 3>, 6);
    case 7: return go(k_soft_mm<true, 3>, 7);
    case 8: return go(k_soft_mm<false, 4>, 8);
    default: return go(k_soft_mm<true, 4>, 9);
    }
}

// ---------------------------------------------------------------------------
// The adjoint for 9 <= N <= 12 dots (formulas at k_soft_bwd), a column per pixel.
// With gl(l) = Gbar . 1_l - Gbar . nb and gc(c) = Gbar . 1_c,
//     ubar(l, c) = -(ikT / Z) F1 F2 W (gl + gc),
// so the sums over its candidates are again products with W and W^T (of F1, F2 and
// of F1 gl, F2 gc: four instead of two), and the sum over the pixels of ubar, which
// dL/dA's pair terms need, is W times the outer products
//     sum_p [(F1 gl / Z) F2^T + (F1 / Z) (F2 gc)^T],
// one more matrix product with the pixels as inner dimension, kept in registers
// (wave w: 16 low states by 64 middle states).  The outer products of dL/dA and
// dL/dC_gd run over the pixels the same way.  Against the walk over the
// candidates, 12 dots and 4096 pixels: 337 -> 23 us.  That is one set of pixels a
// block: a serial chain through eight barriers at one wave a SIMD, where the products
// alone would take 5 us.  (The pair sums at the end had taken 8 us of 36 as a loop
// that waited for each read.)
// ---------------------------------------------------------------------------
template <bool CLOSED>
struct BwdLds {
    static constexpr int kStride = SoftLds<CLOSED>::kStride;
    double F1[kSoftRows][kStride], F2[kSoftRows][kStride];  // factors
    double G1[kSoftRows][kStride], G2[kSoftRows][kStride];  // F1 gl, F2 gc
    double part[4][2][5][kSoftRows];
    double pz[4][kSoftRows];                                // partial normalisers
    double g0[kSoftRows][kMaxDot], gb[kSoftRows][kMaxDot];  // [pixel][dot]
    double z[kSoftRows][kMaxDot + 1], m[kSoftRows][kMaxDot + 1], dx[kSoftRows][kMaxDot + 1];
    double v[kSoftRows][kMaxGate + 2];                      // voltages
    double iz[kSoftRows];                                   // 1 / Z (0 past the last pixel)
    int K[kSoftRows];
    unsigned long long cmin[CLOSED ? 2 : 1][kSoftRows][8];
};

template <bool CLOSED>
__global__ __launch_bounds__(kSoftThreads, 2) void k_soft_mm_bwd(
    const DiagRec *__restrict__ dr, const RowTab *__restrict__ rt, const double *__restrict__ V,
    int64_t P, const double *__restrict__ gbar, const SavedRec *__restrict__ saved,
    double *__restrict__ acc, double *__restrict__ gradV, const VGrid vg)
{
    constexpr int STEPS = SoftLds<CLOSED>::kSteps, STRIDE = SoftLds<CLOSED>::kStride;
    constexpr int CLASSES = CLOSED ? 7 : 1;
    // the table T during the prologue, the batch's buffers, the state sums at the end
    __shared__ union Shared {
        double T[64 * kTStride];
        BwdLds<CLOSED> L;
        struct {
            double low[7][64];  // [all, middle dot 6..11][low state]
            double mid[4][64];  // [wave][middle state]
        } S;
        __device__ Shared() {}
    } sh;
    __shared__ double sA[kMaxDot * kMaxDot], sC[kMaxDot * kMaxGate], sCt[kMaxGate * kMaxDot];
    BwdLds<CLOSED> &L = sh.L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = tid & 15, pix = tid >> 4;  // dot (or gate) and pixel of this thread
    const int q = lane >> 4, col = lane & 15;
    const int n = dr->n, g = dr->g;
    const double ikT = 1.0 / dr->kT;
    const int64_t batches = (P + kSoftRows - 1) / kSoftRows;
    // what a thread (pixel, dot) reads of a batch, one batch ahead: V_d and V_16+d,
    // dL/d<n_d> (0 past the last pixel) and the saved candidate set
    struct In {
        double v0, v1, gb, nb;
        uint32_t fm;
        int k, n0;
    };
    auto fetch = [&](int64_t b) -> In {
        const bool real = b * kSoftRows + pix < P;
        const int64_t p = real ? b * kSoftRows + pix : P - 1;
        In r;
        if (vg.on) {
            double ga, gb;
            grid_ab(vg, p, ga, gb);
            r.v0 = d < g ? grid_v(vg, d, ga, gb) : 0.0;
            r.v1 = 16 + d < g ? grid_v(vg, 16 + d, ga, gb) : 0.0;
        } else {
            r.v0 = d < g ? V[p * g + d] : 0.0;
            r.v1 = 16 + d < g ? V[p * g + 16 + d] : 0.0;
        }
        r.gb = (d < n && real) ? gbar[p * n + d] : 0.0;
        r.nb = saved[p].nb[d];
        r.fm = saved[p].free;
        r.k = saved[p].k;
        r.n0 = saved[p].n0[d];
        return r;
    };
    In next = fetch(blockIdx.x);
    sA[tid] = dr->A[tid];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int e = r * kSoftThreads + tid;
        const double c = dr->Cgd[e];
        sC[e] = c;
        sCt[(e % kMaxGate) * kMaxDot + e / kMaxGate] = c;
    }
    for (int r = 0; r < 16; ++r) {
        const int e = r * kSoftThreads + tid;
        sh.T[(e >> 6) * kTStride + (e & 63)] = (&rt->T[0][0])[e];
    }
    __syncthreads();
    SoftW<STEPS> W;
    soft_w<CLOSED, STEPS>(sh.T, ikT, w, W);
    SoftConst sc;
    soft_const<0>(rt, sh.T, sc);
    __syncthreads();
    for (int i = tid; i < 4 * kSoftRows * STRIDE; i += kSoftThreads)
        (&L.F1[0][0])[i] = 0.0;  // F1, F2, G1, G2: the padding slots stay zero
    f64x4_t U[4] = {};           // middle states 16 i + .., low states 16 w + ..
    f64x4_t out = {};            // wave 0: sum z m^T; waves 1, 2: sum dx V^T
    for (int64_t b = blockIdx.x; b < batches; b += gridDim.x) {
        const int64_t p = b * kSoftRows + pix;
        const bool real = p < P;
        const In in = next;
        if (b + gridDim.x < batches) next = fetch(b + gridDim.x);
        // keep the reads of A and C_gd inside the loop (in registers for the whole
        // kernel they would spill)
        asm volatile("" ::: "memory");
        // x_u = C_gd V by lane = dot
        double xu = 0.0;
        // (C_gd and the voltages are zero past the last gate, z and m past the last dot)
        static_for_dev<0, 16>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            xu += sCt[j * kMaxDot + d] * dppd<kDppRowBcast0 + j>(in.v0);
        });
        if (g > 16)
            static_for_dev<0, 16>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                xu += sCt[(16 + j) * kMaxDot + d] * dppd<kDppRowBcast0 + j>(in.v1);
            });
        const double z = d < n ? (double)in.n0 - xu : 0.0;
        double g0 = 0.0;
        static_for_dev<0, kMaxDot>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            g0 += sA[j * kMaxDot + d] * dppd<kDppRowBcast0 + j>(z);
        });
        const double gnb = row_sum(in.gb * in.nb);
        __syncthreads();  // the last batch's products have read the buffers
        L.g0[pix][d] = g0;
        L.gb[pix][d] = in.gb;
        L.z[pix][d] = z;
        L.v[pix][d] = in.v0;
        L.v[pix][16 + d] = in.v1;
        if (d == 0) L.K[pix] = in.k;
        if constexpr (CLOSED) {
            (&L.cmin[0][0][0])[tid] = ordered(kNoState);
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a pixel's lanes share a wave
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        {
            double f1[4], f2[4];
            soft_factors<CLOSED, 0>(L.g0[pix], in.fm, in.k, sc, ikT, L, f1, f2);
            const double *gb = L.gb[pix];
            double gl = -gnb, gc = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gl = fma(sc.bit[j], gb[j], gl);
                gc = fma(sc.bit[j], gb[6 + j], gc);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = soft_slot<CLOSED>(d + 16 * i);
                const double l = gl + ((i & 1 ? gb[4] : 0.0) + (i & 2 ? gb[5] : 0.0));
                const double c = gc + ((i & 1 ? gb[10] : 0.0) + (i & 2 ? gb[11] : 0.0));
                L.F1[pix][at] = f1[i];
                L.F2[pix][at] = f2[i];
                L.G1[pix][at] = f1[i] * l;
                L.G2[pix][at] = f2[i] * c;
            }
        }
        __syncthreads();
        {
            const int K = CLOSED ? L.K[col] : 0;
            double v[4], vz = 0.0, s5[5];
            f64x4_t a[CLASSES] = {};
            // low states: Z, then G1 Y + F1 (W^T G2)
            soft_product<CLOSED, STEPS, CLASSES>(W.y, &L.F2[0][0], STRIDE, a);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = 16 * w + q + 4 * i, at = soft_slot<CLOSED>(s);
                const double y = soft_pick<CLOSED>(a, i, s, K);
                vz = fma(L.F1[col][at], y, vz);
                v[i] = L.G1[col][at] * y;
            }
#pragma unroll
            for (int m = 0; m < CLASSES; ++m) a[m] = f64x4_t{};
            soft_product<CLOSED, STEPS, CLASSES>(W.y, &L.G2[0][0], STRIDE, a);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = 16 * w + q + 4 * i;
                v[i] = fma(L.F1[col][soft_slot<CLOSED>(s)], soft_pick<CLOSED>(a, i, s, K), v[i]);
            }
            soft_sums5(v, s5);
            vz += other_row(vz);
            vz += other_half(vz);
            if (q == 0) {
#pragma unroll
                for (int j = 0; j < 5; ++j) L.part[w][0][j][col] = s5[j];
                L.pz[w][col] = vz;
            }
            // middle states: G2 X + F2 (W G1)
#pragma unroll
            for (int m = 0; m < CLASSES; ++m) a[m] = f64x4_t{};
            soft_product<CLOSED, STEPS, CLASSES>(W.x, &L.F1[0][0], STRIDE, a);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = 16 * w + q + 4 * i;
                v[i] = L.G2[col][soft_slot<CLOSED>(s)] * soft_pick<CLOSED>(a, i, s, K);
            }
#pragma unroll
            for (int m = 0; m < CLASSES; ++m) a[m] = f64x4_t{};
            soft_product<CLOSED, STEPS, CLASSES>(W.x, &L.G1[0][0], STRIDE, a);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = 16 * w + q + 4 * i;
                v[i] = fma(L.F2[col][soft_slot<CLOSED>(s)], soft_pick<CLOSED>(a, i, s, K), v[i]);
            }
            soft_sums5(v, s5);
            if (q == 0) {
#pragma unroll
                for (int j = 0; j < 5; ++j) L.part[w][1][j][col] = s5[j];
            }
        }
        __syncthreads();
        {
            // thread (pixel, dot): m, dL/dx_u = -A m, dL/dV
            const double Z = (L.pz[0][pix] + L.pz[1][pix]) + (L.pz[2][pix] + L.pz[3][pix]);
            const double iz = real ? 1.0 / Z : 0.0;
            const double md =
                d < n ? -(ikT * iz) * soft_dot_sum(L.part, d >= 6 ? 1 : 0, d >= 6 ? d - 6 : d, pix) : 0.0;
            double dx = 0.0;
            static_for_dev<0, 12>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                dx -= sA[j * kMaxDot + d] * dppd<kDppRowBcast0 + j>(md);
            });
            double gv0 = 0.0, gv1 = 0.0;
            static_for_dev<0, 12>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const double t = dppd<kDppRowBcast0 + j>(dx);
                gv0 += sC[j * kMaxGate + d] * t;
                gv1 += sC[j * kMaxGate + 16 + d] * t;
            });
            if (gradV && real) {
                if (d < g) gradV[p * g + d] = gv0;
                if (16 + d < g) gradV[p * g + 16 + d] = gv1;
            }
            L.m[pix][d] = md;
            L.dx[pix][d] = d < n ? dx : 0.0;
            if (d == 0) L.iz[pix] = iz;
        }
        __syncthreads();
        // sums over the pixels: inner index 4 t + q = pixel
        auto pixel_sums = [&](auto &&keep) {
            static_for_dev<0, 4>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                const int px = 4 * t + q, at = soft_slot<CLOSED>(16 * w + col);
                const double iz = keep(px) ? L.iz[px] : 0.0;
                const double b1 = L.G1[px][at] * iz, b2 = L.F1[px][at] * iz;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int as = soft_slot<CLOSED>(16 * i + col);
                    U[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(L.F2[px][as], b1, U[i], 0, 0, 0);
                    U[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(L.G2[px][as], b2, U[i], 0, 0, 0);
                }
            });
        };
        if constexpr (!CLOSED) {
            pixel_sums([](int) { return true; });
        } else {
            // one sum per raised count among the pixels: its pairs of classes only
            unsigned todo = 0xFFFFu;
            while (todo) {
                const int K = L.K[__builtin_ctz(todo)];
                unsigned same = 0;
                for (int i = 0; i < 16; ++i) same |= L.K[i] == K ? 1u << i : 0u;
                todo &= ~same;
                f64x4_t keep[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { keep[i] = U[i]; U[i] = f64x4_t{}; }
                pixel_sums([&](int px) { return (same >> px & 1u) != 0; });
                const int pl = __popc((uint32_t)(16 * w + col));
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        U[i][e] = pl + __popc((uint32_t)(16 * i + q + 4 * e)) == K ? keep[i][e] + U[i][e]
                                                                                  : keep[i][e];
            }
        }
        if (w < 3) {
            static_for_dev<0, 4>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                const int px = 4 * t + q;
                const double a = w == 0 ? L.z[px][col] : L.dx[px][col];
                const double bb = w == 0 ? L.m[px][col] : L.v[px][16 * (w - 1) + col];
                out = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bb, out, 0, 0, 0);
            });
        }
    }
    // dL/dA also takes half the sums of ubar over the states with dots i and j
    // raised: U times W and -1 / kT, then its sums over the middle states (all, and
    // those with each dot) for every low state, and over the low states
    __syncthreads();
    const int l = 16 * w + col;
    if constexpr (CLOSED) {
        // W in the order of the states: again from the table
        for (int r = 0; r < 16; ++r) {
            const int e = r * kSoftThreads + tid;
            sh.T[(e >> 6) * kTStride + (e & 63)] = (&rt->T[0][0])[e];
        }
        __syncthreads();
        const double tl = sh.T[63 * kTStride + l], tt = 0.25 * sh.T[63 * kTStride + 63];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 16 * i + q + 4 * e;
                const double t = (sh.T[c * kTStride + l] - 0.5 * (tl + sh.T[c * kTStride + 63])) + tt;
                double u = U[i][e] * (-ikT * exp_small(-t * ikT));
                asm volatile("" : "+v"(u));  // (one exponential at a time)
                U[i][e] = u;
            }
        __syncthreads();
    } else {
        // element (i, e): middle state 16 i + q + 4 e = 4 (4 i + e) + q, the lane's own
        // entry of W^T in step 4 i + e
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) U[i][e] *= -ikT * W.y[4 * i + e];
    }
    {
        // over the middle states: bits 4, 5 are i; 2, 3 are e; 0, 1 are q
        double v[4], s5[5], b4 = 0.0, b5 = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = (U[0][e] + U[1][e]) + (U[2][e] + U[3][e]);
            b4 += U[1][e] + U[3][e];
            b5 += U[2][e] + U[3][e];
        }
        soft_sums5(v, s5);
        b4 += other_row(b4);
        b4 += other_half(b4);
        b5 += other_row(b5);
        b5 += other_half(b5);
        if (q == 0) {
#pragma unroll
            for (int j = 0; j < 5; ++j) sh.S.low[j][l] = s5[j];
            sh.S.low[5][l] = b4;
            sh.S.low[6][l] = b5;
        }
        // over the wave's low states
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double t = row_sum(U[i][e]);
                if (col == 0) sh.S.mid[w][16 * i + q + 4 * e] = t;
            }
    }
    // 1/2 (z m^T + m z^T) from wave 0's sum, by way of LDS
    if (w == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e) sA[(q + 4 * e) * kMaxDot + col] = out[e];
    __syncthreads();
    double *accA = acc + (blockIdx.x & (kBwdReplicas - 1)) * kBwdAccWords;
    double *accG = accA + kMaxDot * kMaxDot;
    for (int e = tid; e < n * n; e += kSoftThreads) {
        const int i = e / n, j = e % n;
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        // the states with both dots raised: of the low states' sums (all, or those with
        // the middle dot hi), or of the middle states' sums
        const int need = hi < 6 ? 1 << lo | 1 << hi : (lo < 6 ? 1 << lo : 1 << (lo - 6) | 1 << (hi - 6));
        const double *low = &sh.S.low[hi < 6 ? 0 : (lo < 6 ? hi - 5 : 0)][0];
        double v = 0.0;
        if (lo < 6) {
#pragma unroll 16
            for (int s = 0; s < 64; ++s) {
                const double x = low[s];
                v += (s & need) == need ? x : 0.0;
            }
        } else {
#pragma unroll 16
            for (int s = 0; s < 64; ++s) {
                const double x = (sh.S.mid[0][s] + sh.S.mid[1][s]) + (sh.S.mid[2][s] + sh.S.mid[3][s]);
                v += (s & need) == need ? x : 0.0;
            }
        }
        v = 0.5 * (sA[i * kMaxDot + j] + sA[j * kMaxDot + i]) + 0.5 * v;
        atomicAdd(&accA[i * kMaxDot + j], v);
    }
    if (w == 1 || w == 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = q + 4 * e, j = 16 * (w - 1) + col;
            if (i < n && j < g) atomicAdd(&accG[i * kMaxGate + j], out[e]);
        }
}

hipError_t launch_soft_mm_bwd(const DiagRec *dr, const RowTab *rt, const double *V, int64_t P,
                              const double *gbar, const SavedRec *saved, double *acc,
                              double *gradV, int n_dot, bool closed, hipStream_t s,
                              const VGrid *sweep)
{
    if (n_dot < 9 || n_dot > 12 || !rt) return hipErrorInvalidValue;
    if (P <= 0) return hipSuccess;
    VGrid vg{};
    if (sweep) vg = *sweep;
    const int64_t batches = (P + kSoftRows - 1) / kSoftRows;
    static int cache[2][64];
    auto go = [&](auto kernel, int slot) {
        hipLaunchKernelGGL(kernel, dim3(soft_blocks(kernel, cache[slot], batches)),
                           dim3(kSoftThreads), 0, s, dr, rt, V, P, gbar, saved, acc, gradV, vg);
        return hipGetLastError();
    };
    return closed ? go(k_soft_mm_bwd<true>, 1) : go(k_soft_mm_bwd<false>, 0);
}

// the row tables of a record that holds A, for the adjoint without a forward call
__global__ __launch_bounds__(kWave) void k_row_tab(const DiagRec *__restrict__ dr,
                                                   RowTab *__restrict__ rt)
{
    __shared__ double sA[kMaxDot * kMaxDot];
    for (int i = threadIdx.x; i < kMaxDot * kMaxDot; i += kWave) sA[i] = dr->A[i];
    __syncthreads();
    prep_row_unit(rt, sA, nullptr, dr->n, blockIdx.x < 8 ? (int)blockIdx.x : 24);
}

hipError_t launch_row_tab(const DiagRec *dr, RowTab *rt, hipStream_t s)
{
    hipLaunchKernelGGL(k_row_tab, dim3(9), dim3(kWave), 0, s, dr, rt);
    return hipGetLastError();
}

}  // namespace qa
