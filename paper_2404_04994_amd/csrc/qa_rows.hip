// qa_rows.hip -- FP64 search of the candidate sets of 9 <= N <= 16 dots
// (Sec. 3.2) in bound order.
//
// The candidates n0 + b of a pixel are split into a low part (dots 0..5, 64
// values: one per lane) and a high part (dots 6..N-1, at most 1024 values); a
// row is the 64 states that share a high part c.  With g = A (n0 - x_u),
//     U(n0 + b) - U(n0) = b^T g + 1/2 b^T A b
//                       = [b_lo^T g_lo + 1/2 b_lo^T A_LL b_lo]      (lane)
//                       + [b_hi^T g_hi + 1/2 b_hi^T A_HH b_hi]      (row)
//                       + b_lo^T A_LH b_hi,
// and the last term is a table of the diagram (dots 6..11: 64 x 64 doubles in
// LDS) plus four per-lane constants (dots 12..15), so a row costs a wave one
// LDS read and a handful of FP64 additions for 64 energies.
//
// Minimising over a real-valued low part gives the lower bound of a row,
//     L(b_hi) = K + b_hi^T s + 1/2 b_hi^T S b_hi,  S = (C_dd,HH)^{-1},
// (closed arrays: plus (m - mu - w^T b_hi)^2 / (2 gamma), m the raised low
// dots); S, s and K come from the setup, which gives their derivation.  Sixteen
// bounds per lane are formed in FP32, and rows whose bound lies above the energy
// of the setup's guess (a state of the set) by more than a margin
// (PixRec.slack) are not computed, so every state within 1e-9 of the minimum
// lies in a computed row.
// Six low dots leave about as many rows of 64 states as eight leave rows of
// 256 (host counts on 16-dot diagrams, three seeds each: 4x4 array 8-43 and
// 9-41 per pixel, random capacitances open 10-27 and 13-31, closed 5-10 and
// 6-13).
#include "qa_device.h"

namespace qa {

constexpr int kModeDense = 0, kModePruned = 1, kModeClosed = 2;
constexpr double kBarred = 0x1p1000;  // energy of a state outside the candidate set
constexpr int kRowThreads = 512;  // the 32 KB table is shared by eight waves

__device__ __forceinline__ double readlane_d(double x, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}

// lane L of v = x (wave-uniform)
template <int L>
__device__ __forceinline__ void write_lane(uint32_t &v, uint32_t x)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "n"(L));
}

// The smaller of two numbers, as the hardware forms it: the other one where one is not a
// number.  (fmin puts an instruction before it for every operand that came through
// integer operations, in case it is a signalling NaN, which no result of arithmetic is.)
// The wait is what a lane exchange needs after its source is written, which the compiler
// does not see inside the block.
__device__ __forceinline__ double num_min(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// minimum over the 64 lanes
__device__ __forceinline__ double wave_min_d(double x)
{
    x = num_min(x, dppd<kDppXor1>(x));
    x = num_min(x, dppd<kDppXor2>(x));
    x = num_min(x, dppd<kDppHalfMirror>(x));
    x = num_min(x, dppd<kDppMirror>(x));
    auto swap_min = [&](auto swap) {
        const uint64_t u = (uint64_t)__double_as_longlong(x);
        const auto lo = swap((uint32_t)u), hi = swap((uint32_t)(u >> 32));
        x = num_min(__longlong_as_double((long long)((uint64_t)lo[0] | ((uint64_t)hi[0] << 32))),
                    __longlong_as_double((long long)((uint64_t)lo[1] | ((uint64_t)hi[1] << 32))));
    };
    swap_min([](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
    swap_min([](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
    return x;
}

// Tables of the block (RowTab up to hs, copied as it is) and one pixel record
// per wave.
struct RowLds {
    double T[64][64];
    double lo[4][64], hi[4][64];
    float hs[16][64];
    PixRec rec[kRowThreads / 64];
};
static_assert(offsetof(RowLds, rec) == kRowTabLdsBytes, "copied as it is");
static_assert(kRowTabLdsBytes % (16 * kRowThreads) == 0, "whole rounds of 16 bytes per thread");
static_assert(sizeof(PixRec) == 4 * 64, "a pixel record is one dword per lane");

// What a lane holds of the diagram: its bits and the quadratic forms of the low
// state `lane`, of the high state `lane` over dots 6..11, and over dots 12..15
// for k = lane mod 16.
struct RowConst {
    double bit[6];
    float bitf[6];
    double hlo, hhi, hk;
};

// both of them, every read issued before the first is used (the caller passes a
// barrier before reading the tables)
__device__ __forceinline__ void row_const(const RowTab *__restrict__ rt, RowConst &c, RowLds &t)
{
    const int lane = threadIdx.x & 63;
    constexpr int R = (int)(kRowTabLdsBytes / (16 * kRowThreads));
    const uint4 *src = reinterpret_cast<const uint4 *>(rt);
    uint4 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[r * kRowThreads + threadIdx.x];
    c.hlo = rt->hlo[lane];
    c.hhi = rt->hhi[lane];
    c.hk = rt->hk[lane & 15];
    uint4 *dst = reinterpret_cast<uint4 *>(&t);
#pragma unroll
    for (int r = 0; r < R; ++r) dst[r * kRowThreads + threadIdx.x] = v[r];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        c.bit[i] = (lane >> i & 1) ? 1.0 : 0.0;
        c.bitf[i] = (float)c.bit[i];
    }
}

// LDS writes of a wave made visible to its lanes (requests of one wave are
// served in order; the fences keep the compiler from moving them)
__device__ __forceinline__ void row_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A pixel's record on its way from memory: lane i holds dword i (one load, issued
// a pixel ahead, one register); put() leaves it in the wave's LDS slot, where
// its fields are broadcast reads.
struct RowRec {
    uint32_t dw;
    __device__ __forceinline__ void load(const PixRec *__restrict__ pr, int64_t p)
    {
        dw = reinterpret_cast<const uint32_t *>(pr + p)[threadIdx.x & 63];
    }
    __device__ __forceinline__ void put(PixRec *slot) const
    {
        row_wave_sync();  // the last pixel's reads come first
        reinterpret_cast<uint32_t *>(slot)[threadIdx.x & 63] = dw;
        row_wave_sync();
    }
};

// A pixel's terms: the lane's low part lg, its row part ch (high states
// lane + 64 k, without dots 12..15), the bound's per-lane parts sl and wl and its
// margin, and which high states exist in the pixel's candidate set.
template <int MODE>
struct RowPixel {
    double lg, ch;
    float sl, mu, wl, slack;
    uint32_t free;
    int k, nflo, pcl;
    unsigned long long ok;  // lanes whose bits exist as a high state's dots 6..11

    __device__ __forceinline__ void load(const PixRec *r, const RowConst &c, int n, float sabsS,
                                         float inv2g, const float (&wb)[10], float wabs)
    {
        constexpr bool PRUNED = MODE != kModeDense, CLOSED = MODE == kModeClosed;
        const int lane = threadIdx.x & 63;
        free = PRUNED ? __builtin_amdgcn_readfirstlane(r->free) : 0xFFFFu;
        lg = c.hlo;
        ch = c.hhi;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            // raising a fixed low dot costs 2^500: such a state never wins, the
            // others are exact (a zero bit times the penalty)
            const double gi = (PRUNED && !(free >> i & 1u)) ? 0x1p500 : r->g0[i];
            lg = fma(c.bit[i], gi, lg);
            ch = fma(c.bit[i], r->g0[6 + i], ch);
        }
        // (dots past n: s = 0 in the record)
        sl = r->K;
        wl = 0.0f;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            sl = fmaf(c.bitf[j], r->s[j], sl);
            if (CLOSED) wl = fmaf(c.bitf[j], wb[j], wl);
        }
        ok = n >= 12 ? ~0ull : (1ull << (1 << (n - 6))) - 1;
        if (PRUNED) ok &= __ballot(!((uint32_t)lane & ~(free >> 6) & 63u));
        pcl = __popc((uint32_t)lane);
        slack = r->slack + 0x1p-19f * sabsS;
        if (CLOSED) {
            k = __builtin_amdgcn_readfirstlane(r->k);
            nflo = __popc(free & 63u);
            mu = r->mu;
            const float lsum = 6.0f + fabsf(mu) + wabs;
            slack += 0x1p-19f * lsum * lsum * inv2g;
        }
    }

    // Which rows may hold a state at or below thr: lane k of (mlo, mhi) receives
    // the mask of the high states .. + 64 k, k < 2^(n - 12); returns the k with
    // any.  A bound that is not a number passes.
    __device__ __forceinline__ uint32_t rows(const PixRec *r, const RowLds &t, int n, float thr,
                                             float inv2g, const float (&wb)[10], uint32_t &mlo,
                                             uint32_t &mhi) const
    {
        constexpr bool PRUNED = MODE != kModeDense, CLOSED = MODE == kModeClosed;
        const int lane = threadIdx.x & 63;
        uint32_t kset = 0;
        float lb[16], W[16];
        mlo = mhi = 0;
        auto part = [&](auto kc) {
            constexpr int KK = decltype(kc)::value;
            if constexpr (KK == 0) {
                lb[0] = sl;
                W[0] = wl;
            } else {
                constexpr int low = KK & (KK - 1), j = __builtin_ctz(KK);
                lb[KK] = lb[low] + r->s[6 + j];
                if (CLOSED) W[KK] = W[low] + wb[6 + j];
            }
            if (PRUNED && ((uint32_t)KK & ~(free >> 12) & 15u)) return;
            float L = lb[KK] + t.hs[KK][lane];
            unsigned long long in = ok;
            if (CLOSED) {
                const int m = k - pcl - __builtin_popcount(KK);
                const float dm = ((float)m - mu) - W[KK];
                L = fmaf(dm * dm, inv2g, L);
                in &= __builtin_amdgcn_uicmp((uint32_t)m, (uint32_t)nflo, 37);  // 0 <= m <= nflo
            }
            const unsigned long long mask = in & __builtin_amdgcn_fcmpf(L, thr, 13);  // not above
            write_lane<KK>(mlo, (uint32_t)mask);
            write_lane<KK>(mhi, (uint32_t)(mask >> 32));
            kset |= mask ? 1u << KK : 0u;
        };
        static_for_dev<0, 1>(part);
        if (n > 12) {
            static_for_dev<1, 2>(part);
            if (n > 13) {
                static_for_dev<2, 4>(part);
                if (n > 14) {
                    static_for_dev<4, 8>(part);
                    if (n > 15) static_for_dev<8, 16>(part);
                }
            }
        }
        return kset;
    }

    // The smallest energy of the row with the lowest bound (kBarred when there is none)
    // of a dense box.  A bound that is not a number is never the lowest.
    __device__ __forceinline__ double lowest(const PixRec *r, const RowConst &c, const RowLds &t,
                                             int n) const
    {
        const int lane = threadIdx.x & 63;
        float best = 0x1p120f;
        int at = 0;
#pragma unroll 1
        for (int kk = 0; kk < 1 << (n > 12 ? n - 12 : 0); ++kk) {
            float L = sl + t.hs[kk][lane];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (kk >> j & 1) L += r->s[6 + j];
            if ((ok >> lane & 1u) && L < best) { best = L; at = kk; }
        }
        float low = best;
        for (int off = 32; off >= 1; off >>= 1) low = fminf(low, __shfl_xor(low, off));
        const unsigned long long hit = __ballot(best == low && best < 0x1p120f);
        if (!hit) return kBarred;
        const int c6 = __builtin_ctzll(hit), kk = __builtin_amdgcn_readlane(at, c6);
        double base = lg, rc = ch + readlane_d(c.hk, kk);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (kk >> j & 1) {
                base += t.lo[j][lane];
                rc += t.hi[j][lane] + r->g0[12 + j];
            }
        return wave_min_d((base + readlane_d(rc, c6)) + t.T[c6][lane]);
    }

    // the energies of those rows (relative to U(n0); kBarred outside a closed set,
    // above 2^499 where a fixed dot is raised): to(row, energy of the lane's state), or two
    // rows at once
    template <bool FOUR, typename To>
    __device__ __forceinline__ void scan(const PixRec *r, const RowConst &c, const RowLds &t,
                                         uint32_t kset, uint32_t mlo, uint32_t mhi, To &to) const
    {
        constexpr bool CLOSED = MODE == kModeClosed;
        const int lane = threadIdx.x & 63;
        for (uint32_t ks = kset; ks; ks &= ks - 1) {
            const int kk = __builtin_ctz(ks);
            unsigned long long mask =
                (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mlo, kk) |
                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mhi, kk) << 32);
            double base = lg, rc = ch + readlane_d(c.hk, kk);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (kk >> j & 1) {
                    base += t.lo[j][lane];
                    rc += t.hi[j][lane] + r->g0[12 + j];
                }
            const int left = k - __popc((uint32_t)kk);  // closed: raised in c6 and the low part
            auto energy = [&](int c6, double tt) {
                const double e = (base + readlane_d(rc, c6)) + tt;
                if (!CLOSED) return e;
                return pcl == left - __popc((uint32_t)c6) ? e : kBarred;
            };
            // Four rows at a time, then two: their table reads and sums overlap.  (A wave
            // that is left alone with hundreds of rows waits for each step; the second
            // pass over ties stays at two for its registers.)
            while (FOUR && __popcll(mask) >= 4) {
                const int c0 = __builtin_ctzll(mask);
                mask ^= 1ull << c0;
                const int c1 = __builtin_ctzll(mask);
                mask ^= 1ull << c1;
                const int c2 = __builtin_ctzll(mask);
                mask ^= 1ull << c2;
                const int c3 = __builtin_ctzll(mask);
                mask ^= 1ull << c3;
                const double t0 = t.T[c0][lane], t1 = t.T[c1][lane];
                const double t2 = t.T[c2][lane], t3 = t.T[c3][lane];
                const double e0 = energy(c0, t0), e1 = energy(c1, t1);
                const double e2 = energy(c2, t2), e3 = energy(c3, t3);
                to(kk * 64 + c0, e0, kk * 64 + c1, e1);
                to(kk * 64 + c2, e2, kk * 64 + c3, e3);
            }
            while (mask & (mask - 1)) {
                const int c0 = __builtin_ctzll(mask);
                mask ^= 1ull << c0;
                const int c1 = __builtin_ctzll(mask);
                mask ^= 1ull << c1;
                const double t0 = t.T[c0][lane], t1 = t.T[c1][lane];
                const double e0 = energy(c0, t0), e1 = energy(c1, t1);
                to(kk * 64 + c0, e0, kk * 64 + c1, e1);
            }
            if (mask) {
                const int c0 = __builtin_ctzll(mask);
                to(kk * 64 + c0, energy(c0, t.T[c0][lane]));
            }
        }
    }
};

// A lane's two smallest energies, the row in the low ten bits of the mantissa.  The
// comparisons are the hardware's, which take the other operand where one is not a number;
// fmin and fmax put an instruction before them for an energy whose low bits were
// replaced, in case it is a signalling NaN (no result of arithmetic is).
struct RowMins {
    double m1 = kBarred, m2 = kBarred;
    uint32_t keep;
    __device__ __forceinline__ double coded(int row, double e) const
    {
        const uint64_t u = (uint64_t)__double_as_longlong(e);
        const uint32_t lo = ((uint32_t)u & keep) | (uint32_t)row;
        return __longlong_as_double((long long)((u & 0xFFFFFFFF00000000ull) | lo));
    }
    static __device__ __forceinline__ double lower(double a, double b)
    {
        double r;
        asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
        return r;
    }
    static __device__ __forceinline__ double upper(double a, double b)
    {
        double r;
        asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
        return r;
    }
    __device__ __forceinline__ void operator()(int row, double e)
    {
        const double x = coded(row, e), t = upper(m1, x);
        m1 = lower(m1, x);
        m2 = lower(m2, t);
    }
    __device__ __forceinline__ void operator()(int row0, double e0, int row1, double e1)
    {
        const double x = coded(row0, e0), y = coded(row1, e1);
        const double lo = lower(x, y), hi = upper(x, y);
        m2 = lower(m2, hi);
        const double t = upper(m1, lo);
        m1 = lower(m1, lo);
        m2 = lower(m2, t);
    }
};

// The same with the energies as they are and the lexicographically smallest state of the
// smallest energy (as brev(state)).
struct RowTies {
    double b1 = kBarred, b2 = kBarred;
    uint32_t best = 0xFFFFFFFFu;
    __device__ __forceinline__ void operator()(int row, double e)
    {
        const uint32_t at = __brev((threadIdx.x & 63) | ((uint32_t)row << 6));
        if (e < b1 || (e == b1 && at < best)) { b2 = b1; b1 = e; best = at; }
        else b2 = fmin(b2, e);
    }
    __device__ __forceinline__ void operator()(int row0, double e0, int row1, double e1)
    {
        (*this)(row0, e0);
        (*this)(row1, e1);
    }
};

// Wave priority by the wave's remaining work: the kernel ends with the waves
// whose pixels take many rows (lane k of mlo, mhi: the rows of k) and with those
// that still hold a pixel after this one, so those waves issue first.
__device__ __forceinline__ void row_priority(uint32_t mlo, uint32_t mhi, bool more)
{
    const bool many = __ballot(__popc(mlo) + __popc(mhi) >= 8) != 0;
    if (many && more) __builtin_amdgcn_s_setprio(3);
    else if (many) __builtin_amdgcn_s_setprio(2);
    else if (more) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// rows in the masks of rows(), held by lanes 0..15
__device__ __forceinline__ int row_count(uint32_t mlo, uint32_t mhi)
{
    int v = __popc(mlo) + __popc(mhi);
    v += (int)dpp32<kDppXor1>((uint32_t)v);
    v += (int)dpp32<kDppXor2>((uint32_t)v);
    v += (int)dpp32<kDppHalfMirror>((uint32_t)v);
    v += (int)dpp32<kDppMirror>((uint32_t)v);
    return __builtin_amdgcn_readfirstlane(v);
}

// From this many rows on, the row with the lowest bound is computed first, and the
// rows are chosen again by its minimum if that is below the guess: some 250
// instructions, a row is 12.  On arrays the kernel's tail are pixels with a poor guess:
// over 1500 pixels of a 16-dot array up to 686 rows by the guess, 84 by this row and
// 68 by the minimum itself (random capacitances: 231, 231 and 218, the bound is loose).
// The form with this step (TAIL) is for dense boxes of 14 dots and more and few pixels,
// where the kernel ends with such pixels; from some number of pixels on all pixels'
// instructions count.  Without / with it, us a call, means over six arrays and six sets
// of random capacitances:
//     16 dots  10^4 37.4 / 32.7, 45.0 / 42.5; 2.5*10^4 60.2 / 55.0, 63.9 / 63.1;
//              5*10^4 89.6 / 88.2, 95.7 / 100.4
//     14 dots  10^4 23.8 / 23.1, 24.9 / 25.2; 2.5*10^4 39.6 / 39.7, 40.7 / 42.2
//     12 dots  10^4 19.1 / 19.2, 18.6 / 18.8; 9 dots 16.9 / 17.3, 16.6 / 17.1
// Thresholded sets are slower with it throughout (16 dots, 10^4 pixels, t = 1/2 34.3 /
// 40.7 random, 30.0 / 34.0 arrays: their guess is not what leaves the rows).
constexpr int kManyRows = 64;
constexpr int64_t kTailPixels = 12500;  // per dot above 13

// T = 0 argmin (Eq. argmin) over each pixel's candidate set: a wave per pixel,
// one lane per low state, over the rows the bound leaves.  Each lane keeps its
// two smallest energies with the row in the low ten bits of the mantissa (an
// error below 2^-42 of the energy, so one minimum carries both).  Where a runner-up
// lies within 1e-9, or within what the row numbers may have changed, the rows are
// taken once more with the energies as they are: the smallest, ties to the
// lexicographically smallest state; a gap below 1e-9 is counted.
template <int MODE, bool TAIL>
__global__ __launch_bounds__(kRowThreads, MODE == kModeClosed ? 4 : 6) void k_rows_gs(const RowTab *__restrict__ rt,
                                                            const PixRec *__restrict__ pr, int64_t P,
                                                            int32_t *__restrict__ n_out, int n,
                                                            int64_t *__restrict__ counters)
{
    constexpr bool PRUNED = MODE != kModeDense, CLOSED = MODE == kModeClosed;
    __shared__ RowLds T;
    __shared__ unsigned long long sc[3];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t nwaves = (int64_t)gridDim.x * (kRowThreads / 64);
    int64_t p = (int64_t)blockIdx.x * (kRowThreads / 64) + wv;
    RowRec next;
    next.load(pr, p < P ? p : P - 1);
    RowConst c;
    row_const(rt, c, T);
    const float sabsS = rt->sabsS, inv2g = CLOSED ? rt->inv2g : 0.0f;
    float wb[10], wabs = 0.0f;
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        wb[j] = CLOSED ? rt->wB[j] : 0.0f;
        wabs += fabsf(wb[j]);
    }
    if (threadIdx.x < 3) sc[threadIdx.x] = 0;
    __syncthreads();
    // (a wave takes at most 2^31 / 6144 pixels, a lane holds at most 64 rows of one)
    int32_t ngap = 0, nrows = 0;
    int64_t ncand = 0;
    const PixRec *r = &T.rec[wv];
    uint32_t keep = ~1023u;
    asm("" : "+v"(keep));  // a register: with a literal the and-or is two instructions
    for (; p < P; p += nwaves) {
        next.put(&T.rec[wv]);
        if (p + nwaves < P) next.load(pr, p + nwaves);
        RowPixel<MODE> px;
        px.load(r, c, n, sabsS, inv2g, wb, wabs);
        if (MODE == kModePruned) ncand += 1ll << __popc(px.free & ((1u << n) - 1u));
        if (CLOSED) ncand += closed_states(__popc(px.free & ((1u << n) - 1u)), px.k);
        uint32_t mlo, mhi;
        uint32_t kset;
        if constexpr (!TAIL) {
            kset = px.rows(r, T, n, r->eg + px.slack, inv2g, wb, mlo, mhi);
        } else {
            float thr = r->eg + px.slack;
#pragma unroll 1
            for (bool again = true;; again = false) {
                kset = px.rows(r, T, n, thr, inv2g, wb, mlo, mhi);
                if (!again || row_count(mlo, mhi) < kManyRows) break;
                const float e = (float)px.lowest(r, c, T, n);
                nrows += lane == 0;
                if (!(e < r->eg)) break;
                thr = e + px.slack + 0x1p-22f * fabsf(e);
            }
        }
        nrows += __popc(mlo) + __popc(mhi);  // (a lane's share: summed at the end)
        row_priority(mlo, mhi, p + nwaves < P);
        RowMins mins;
        mins.keep = keep;
        px.template scan<PRUNED || TAIL>(r, c, T, kset, mlo, mhi, mins);
        const double m1 = mins.m1, m2 = mins.m2;
        const double e1 = wave_min_d(m1);
        const unsigned long long hit = __ballot(m1 == e1);
        const int win = hit ? __builtin_ctzll(hit) : 0;
        const uint32_t code = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)__double_as_longlong(e1));
        uint32_t s = (e1 < 0x1p499) ? (uint32_t)win | ((code & 1023u) << 6) : 0u;
        // a runner-up that may be nearer than 1e-9 or the smaller one (both energies are
        // off by 2^-42 of themselves): another lane's best or some lane's second
        const double near = fma(0x1p-40, fabs(e1), e1 + 2e-9);
        if (__popcll(__ballot(m1 < near)) > 1 || __ballot(m2 < near)) {
            RowTies ties;
            px.template scan<false>(r, c, T, kset, mlo, mhi, ties);
            double b1 = ties.b1, b2 = ties.b2;
            uint32_t best = ties.best;
            for (int off = 32; off >= 1; off >>= 1) {
                const double o1 = __shfl_xor(b1, off), o2 = __shfl_xor(b2, off);
                const uint32_t oa = __shfl_xor(best, off);
                if (o1 < b1 || (o1 == b1 && oa < best)) { b2 = fmin(b1, o2); b1 = o1; best = oa; }
                else b2 = fmin(b2, o1);
            }
            if (b1 < 0x1p499) s = __brev(best);
            if (b1 < 0x1p499 && b2 - b1 < 1e-9) ++ngap;
        }
        if (lane < n) n_out[p * n + lane] = r->n0[lane & 15] + (int32_t)(s >> lane & 1u);
    }
    const int64_t rows = (int64_t)wave_sum((double)nrows);
    if (lane == 0) {
        if (ngap) atomicAdd(&sc[0], (unsigned long long)ngap);
        if (rows) atomicAdd(&sc[1], (unsigned long long)rows);
        if (ncand) atomicAdd(&sc[2], (unsigned long long)ncand);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        block_add_counter(counters, C_GAP_1E9, (int64_t)sc[0]);
        block_add_counter(counters, C_SCORED, (int64_t)sc[1] << 6);
        if (PRUNED) block_add_counter(counters, C_CANDIDATES, (int64_t)sc[2]);
        else if (blockIdx.x == 0) block_add_counter(counters, C_CANDIDATES, P << n);
    }
}

// blocks of a row kernel that fit on the device at once (cached per device)
template <typename Kernel>
static int64_t row_blocks(Kernel kernel, int (&cache)[64], int64_t P)
{
    const int64_t all = (P + kRowThreads / 64 - 1) / (kRowThreads / 64);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return all;
    if (!cache[dev]) {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kRowThreads, 0) != hipSuccess ||
            per_cu <= 0)
            return all;
        cache[dev] = cus * per_cu;
    }
    return all < cache[dev] ? all : cache[dev];
}

hipError_t launch_rows_gs(const RowTab *rt, const PixRec *pr, int64_t P, int mode, int32_t *n_out,
                          int64_t *counters, int n_dot, hipStream_t s)
{
    if (n_dot < 9 || n_dot > kMaxDot || mode < kModeDense || mode > kModeClosed)
        return hipErrorInvalidValue;
    if (P <= 0) return hipSuccess;
    static int cache[4][64];
    auto go = [&](auto kernel, int slot) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)row_blocks(kernel, cache[slot], P)),
                           dim3(kRowThreads), 0, s, rt, pr, P, n_out, n_dot,
                           counters);
        return hipGetLastError();
    };
    if (mode == kModeDense)
        return P <= kTailPixels * (n_dot - 13) ? go(k_rows_gs<kModeDense, true>, 3)
                                : go(k_rows_gs<kModeDense, false>, mode);
    if (mode == kModePruned) return go(k_rows_gs<kModePruned, false>, mode);
    return go(k_rows_gs<kModeClosed, false>, mode);
}

}  // namespace qa
