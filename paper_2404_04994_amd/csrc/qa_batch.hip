// qa_batch.hip -- a ragged batch of stability diagrams (different dot counts,
// open and closed arrays, different temperatures) in two launches,
// the dataset-generation use the paper motivates (Sec. 1, Sec. 8).
//
//   k_prep_batch  one block per diagram: copies C_dd, C_gd and the solve
//                 mode into a DiagRec and runs the same prologue as a single
//                 diagram (A = C_dd^{-1} in FP64); notes the diagram that owns
//                 each work item and clears the counters.
//   k_batch       a wave per work item of 64 pixels of one diagram, so every
//                 lane of the wave shares its dot count and candidate layout.
//                 Lane = pixel, and the whole path runs in registers: x_u =
//                 C_gd V, the analytic minimum or the exact QP (Sec. 3.1), the
//                 candidate set (Sec. 3.2), the argmin (Eq. argmin) and, when
//                 kT > 0, the softargmin (Eq. softargmin) over the set, all
//                 energies in FP64.  Nothing per pixel goes back to HBM except
//                 the results.
#include "qa_device.h"

namespace qa {

__global__ __launch_bounds__(kPrepThreads) void k_prep_batch(const BatchHdr *__restrict__ hdr,
                                                   const double *__restrict__ mats,
                                                   DiagRec *__restrict__ recs,
                                                   int32_t *__restrict__ owner,
                                                   int64_t *__restrict__ counters)
{
    __shared__ double sCdd[kMaxDot * kMaxDot];
    __shared__ double M[kMaxDot * kMaxDot];
    __shared__ double cvec[kMaxDot];
    __shared__ double red[8];
    const BatchHdr h = hdr[blockIdx.x];
    DiagRec *dr = recs + blockIdx.x;
    // (by the first block alone: an index over the grid passes 2^31 from 2^23 diagrams on)
    if (blockIdx.x == 0)
        for (int e = threadIdx.x; e < kCounterWords; e += kPrepThreads) counters[e] = 0;
    const int64_t items = (h.P + 63) / 64;
    for (int64_t e = threadIdx.x; e < items; e += kPrepThreads)
        owner[h.tile0 + e] = blockIdx.x;
    const int n = h.n, g = h.g;
    const double *cdd = mats + h.mat_off;
    const double *cgd = cdd + n * n;
    // (all reads, one round trip, then the stores; C_dd stays in LDS for the inverse)
    static_assert(kPrepThreads == kMaxDot * kMaxDot && 2 * kPrepThreads == kMaxDot * kMaxGate,
                  "an entry of C_dd and two of C_gd a thread");
    const int e = threadIdx.x;
    const int ci = e / kMaxDot, cj = e % kMaxDot, gi = e / kMaxGate, gj = e % kMaxGate;
    const double c = ci < n && cj < n ? cdd[ci * n + cj] : 0.0;
    const double g0 = gi < n && gj < g ? cgd[gi * g + gj] : 0.0;
    const double g1 = 8 + gi < n && gj < g ? cgd[(8 + gi) * g + gj] : 0.0;
    sCdd[e] = c;
    dr->Cdd[e] = c;
    dr->Cgd[e] = g0;
    dr->Cgd[kPrepThreads + e] = g1;
    if (threadIdx.x == 0) {
        dr->n = n;
        dr->g = g;
        dr->closed = h.closed;
        dr->nhat = h.nhat;
        dr->kT = h.kT;
        dr->t = h.t;
        dr->prec = 0;
    }
    __syncthreads();
    prep_inverse(sCdd, n, M, cvec, red);
    prep_store(dr, M, cvec, red, n);
}

hipError_t launch_prep_batch(const BatchHdr *hdr, const double *mats, DiagRec *recs, int n_diag,
                             int32_t *owner, int64_t *counters, hipStream_t s)
{
    hipLaunchKernelGGL(k_prep_batch, dim3(n_diag), dim3(kPrepThreads), 0, s, hdr, mats, recs,
                       owner, counters);
    return hipGetLastError();
}

// Dense box of n <= 8 dots (every dot free), walked by one lane.  With s the
// raised dots and h(s) = 1/2 s^T A s from the diagram's table (LDS),
//     U(n0 + s) - U(n0) = s . g0 + h(s)                       (Eq. free_energy)
// The 2^n states are visited in blocks of sixteen Gray-code steps: inside a
// block only dots 0..3 flip, the flipped dot and (for dots 0..2) its new value
// are compile-time constants, and gray(16 o + k) = gray(16 o) ^ gray(k).
// Pass 1 finds the smallest and the second smallest energy; pass 2 finds the
// lexicographically smallest state at the smallest one (the rank brev(s)) and,
// for kT > 0, the Boltzmann sums (weights by the hardware exp2 in FP32 of
// an FP64 argument, relative error below 3e-6 for every weight above e^-60;
// sums in FP64).
//
// Both passes leave out the blocks whose energies are all above what they look
// for in every pixel of the wave.  A block's high dots give the bound
//     min_lo U >= L_hi + h(hi) + sum_{i<4} min(0, g0_i + h(hi + 1_i) - h(hi)) - neg,
// neg = the sum of the negative A_ij, i < j < 4 (none for a capacitance matrix).
// Pass 1 compares it with the smallest energy so far (at the start that of x*
// rounded), pass 2 with e1 + 87.4 kT, past which the FP32 weights are zero.
struct BlockBound {
    double hd[16][4];  // h(hi + 1_i) - h(hi)
    double neg;        // sum of max(0, -A_ij), i < j < 4
    double hmax;       // 1/2 sum |A_ij|: bounds every h
};

// What a tile reads of its diagram, in LDS.  (As scalar loads from the record
// these had been the longest part of a tile: a tile of C_gd, A and, each round of
// the QP, C_dd, in pieces that fit the scalar registers, each a miss of the scalar
// cache, which two CUs' waves share with a diagram each.)
template <int NM>
struct DiagLds {
    double A[NM * kMaxDot];
    double K[NM * kMaxDot];     // the QP's matrix (qp_solve)
    double Cgt[kMaxGate * NM];  // [gate][dot]
    double c[NM];
    double hs[NM <= 8 ? 256 : 1];
    BlockBound bb;
};

template <int NM, bool CLOSED>
__device__ __forceinline__ void dense_small(const double *__restrict__ sh,
                                            const BlockBound &bb, const double (&g0)[NM],
                                            const double (&x)[NM], const int (&n0)[NM], int n,
                                            int k, double kT, bool soft, double &e1out,
                                            double &e2out, uint32_t &s1out, double &Z,
                                            double (&sv)[NM])
{
    const int nb = n > 4 ? 1 << (n - 4) : 1;
    // the bound of block o against the lane's threshold
    auto skip = [&](uint32_t hi, double Lhi, int pchi, double thr) {
        double lb = Lhi + sh[hi];
#pragma unroll
        for (int i = 0; i < 4; ++i) lb += fmin(0.0, g0[i] + bb.hd[hi >> 4][i]);
        bool out = lb - bb.neg > thr;
        if (CLOSED) out |= (unsigned)(k - pchi) > 4u;
        return !__any(!out);
    };
    // every state of block o: visit(e, gk), e = infinity for those without k raised dots
    auto block = [&](uint32_t sb, int par, int pchi, double L, auto &&visit) {
        const double *ha = sh + sb, *hb = sh + (sb ^ 8u);
        const int ka = k - pchi - par, kb = k - pchi - 1 + par;
        auto steps = [&](auto first, auto last) {
            static_for_dev<decltype(first)::value, decltype(last)::value>([&](auto kc) {
                constexpr int kk = decltype(kc)::value;
                constexpr uint32_t gk = (uint32_t)(kk ^ (kk >> 1));
                if constexpr (kk > 0) {
                    constexpr int d = __builtin_ctz(kk);
                    if constexpr (d < 3) L += ((gk >> d) & 1u) ? g0[d] : -g0[d];
                    else L += par ? -g0[3] : g0[3];
                }
                double e = L + (gk & 8u ? hb[gk & 7u] : ha[gk & 7u]);
                if (CLOSED)
                    e = (gk & 8u ? kb : ka) == __builtin_popcount(gk & 7u) ? e : INFINITY;
                visit(e, std::integral_constant<uint32_t, gk>{});
            });
        };
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, 2> c2{};
        constexpr std::integral_constant<int, 4> c4{};
        constexpr std::integral_constant<int, 8> c8{};
        constexpr std::integral_constant<int, 16> c16{};
        steps(c0, c2);
        if (n < 2) return;
        steps(c2, c4);
        if (n < 3) return;
        steps(c4, c8);
        if (n < 4) return;
        steps(c8, c16);
    };
    auto high = [&](uint32_t sb) {
        double L = 0.0;
#pragma unroll
        for (int i = 0; i < NM; ++i)
            if (sb >> i & 1u) L += g0[i];
        return L;
    };
    double e1 = INFINITY, e2 = INFINITY;
    double thr = INFINITY, slack = 0.0;
    if (nb > 1) {
        uint32_t sr = 0;
        if (CLOSED) {
            // the k largest parts x - n0 raised
            int rank[NM] = {};
#pragma unroll
            for (int i = 1; i < NM; ++i)
#pragma unroll
                for (int j = 0; j < i; ++j) {
                    const bool gt = x[i] - n0[i] > x[j] - n0[j];
                    rank[i] += gt ? 0 : 1;
                    rank[j] += gt ? 1 : 0;
                }
#pragma unroll
            for (int i = 0; i < NM; ++i) sr |= rank[i] < k ? 1u << i : 0u;
            sr &= (1u << n) - 1u;
        } else {
#pragma unroll
            for (int i = 0; i < NM; ++i) sr |= x[i] - n0[i] > 0.5 ? 1u << i : 0u;
        }
        double L = 0.0, sa = 0.0;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            L += sr >> i & 1u ? g0[i] : 0.0;
            sa += fabs(g0[i]);
        }
        // rounding of the bound and of the energies, and room for the gap's 1e-9
        slack = 2e-9 + 1e-13 * (sa + bb.hmax);
        if (!CLOSED || __popc(sr) == k) thr = L + sh[sr] + slack;
    }
    for (int o = 0; o < nb; ++o) {
        const uint32_t sb = ((uint32_t)o << 4) ^ ((uint32_t)o << 3);
        const int par = o & 1, pchi = __popc(sb >> 4);
        const double L = high(sb);
        if (nb > 1 && skip(sb & ~15u, high(sb & ~15u), pchi, thr)) continue;
        block(sb, par, pchi, L, [&](double e, auto) {
            e2 = fmin(e2, fmax(e1, e));
            e1 = fmin(e1, e);
        });
        thr = fmin(thr, e1 + slack);
    }
    const double c = soft ? 1.4426950408889634 / kT : 0.0;
    uint32_t r1 = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < NM; ++i) sv[i] = 0.0;
    Z = 0.0;
    thr = e1 + slack + (soft ? 87.4 * kT : 0.0);
    for (int o = 0; o < nb; ++o) {
        const uint32_t sb = ((uint32_t)o << 4) ^ ((uint32_t)o << 3);
        const uint32_t rb = __brev(sb);
        const int par = o & 1, pchi = __popc(sb >> 4);
        const double L = high(sb);
        if (nb > 1 && skip(sb & ~15u, high(sb & ~15u), pchi, thr)) continue;
        float sblk = 0.0f, t0 = 0.0f, t1 = 0.0f, t2 = 0.0f, t3 = 0.0f;
        if (soft) {
            block(sb, par, pchi, L, [&](double e, auto gc) {
                constexpr uint32_t gk = decltype(gc)::value;
                r1 = min(r1, e == e1 ? rb ^ __builtin_bitreverse32(gk) : 0xFFFFFFFFu);
                const float w = __builtin_amdgcn_exp2f((float)((e1 - e) * c));
                sblk += w;
                if constexpr (gk & 1u) t0 += w;
                if constexpr (gk & 2u) t1 += w;
                if constexpr (gk & 4u) t2 += w;
                if constexpr (gk & 8u) t3 += w;
            });
            Z += sblk;
            sv[0] += t0;
            if (NM > 1) sv[1] += t1;
            if (NM > 2) sv[2] += t2;
            if (NM > 3) sv[3] += par ? (double)(sblk - t3) : (double)t3;
#pragma unroll
            for (int i = 4; i < NM; ++i)
                if (sb >> i & 1u) sv[i] += sblk;
        } else {
            block(sb, par, pchi, L, [&](double e, auto gc) {
                constexpr uint32_t gk = decltype(gc)::value;
                r1 = min(r1, e == e1 ? rb ^ __builtin_bitreverse32(gk) : 0xFFFFFFFFu);
            });
        }
    }
    e1out = e1;
    e2out = e2;
    // (no state below infinity: voltages that are not numbers)
    s1out = e1 < INFINITY ? __brev(r1) : 0xFFFFFFFFu;
}

// one pixel, lane-sequential: returns the size of its candidate set
// (xu: x_u = C_gd V)
template <int NM>
__device__ __forceinline__ int64_t batch_pixel(const DiagLds<NM> &L, const BatchHdr &h,
                                               double one_c,
                                               const double (&xu)[NM],
                                               int32_t *__restrict__ nout,
                                               double *__restrict__ nbout, int &qp, int &fail,
                                               int &dbl, int &gap)
{
    const int n = h.n;
    const bool closed = h.closed != 0;
    const double nhat = (double)h.nhat;
    double x[NM];
    // analytic minimum first (Sec. 3.1.1), the QP only when it is negative
    double lam = 0.0;
    if (closed) {
        double sx = 0.0;
#pragma unroll
        for (int i = 0; i < NM; ++i) sx += xu[i];
        lam = (nhat - sx) / one_c;
    }
    bool feasible = true;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        x[i] = (i < n) ? xu[i] + lam * L.c[i] : 0.0;
        feasible &= x[i] >= 0.0;
    }
    if (closed && h.nhat == 0) {
        qp = !feasible;
#pragma unroll
        for (int i = 0; i < NM; ++i) x[i] = 0.0;
        feasible = true;
    }
    if (!feasible) {
        qp = 1;
        double scale = 1.0, x0[NM];
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            scale = fmax(scale, fabs(xu[i]));
            x0[i] = x[i];
        }
        const double tol = 1e-13 * scale;
        bool ok = false;
        if constexpr (NM <= 8) {
            // the QP at the diagram's own size (its factorisation is cubic in
            // the order; dots n.. of x are zero already).  The rest of the
            // path stays at NM: one copy of it per dot count made the kernel
            // too large for the instruction cache.
            static_for_dev<1, NM + 1>([&](auto kc) {
                constexpr int K = decltype(kc)::value;
                if (n == K)
                    ok = qp_solve<K>(L.K, tol, *reinterpret_cast<const double(*)[K]>(&x0[0]),
                                     *reinterpret_cast<double(*)[K]>(&x[0]));
            });
        } else {
            ok = qp_solve<NM>(L.K, tol, x0, x);
        }
        fail = ok ? 0 : 1;
    }
    int n0[NM];
    uint32_t fm;
    int k;
    const int flags = candidate_set<NM>(n, closed, h.nhat, h.t, x, n0, fm, k);
    dbl = (flags & 4) ? 1 : 0;
    double g0[NM];
    double u0 = 0.0;
    if constexpr (NM <= 8) {
        // at the diagram's own size too (quadratic in it; the padding of A
        // adds zeros only)
#pragma unroll
        for (int i = 0; i < NM; ++i) g0[i] = 0.0;
        static_for_dev<1, NM + 1>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            if (n == K)
                u0 = base_state<K>(L.A, n, *reinterpret_cast<const int(*)[K]>(&n0[0]),
                                   *reinterpret_cast<const double(*)[K]>(&xu[0]),
                                   *reinterpret_cast<double(*)[K]>(&g0[0]));
        });
    } else {
        u0 = base_state<NM>(L.A, n, n0, xu, g0);
    }
    if (NM <= 8 && fm == (1u << n) - 1u) {
        // dense box: table-driven walk
        const bool soft = nbout != nullptr && h.kT > 0.0;
        double e1, e2, Z, sv[NM];
        uint32_t s1;
        if (closed)
            dense_small<NM, true>(L.hs, L.bb, g0, x, n0, n, k, h.kT, soft, e1, e2, s1, Z, sv);
        else
            dense_small<NM, false>(L.hs, L.bb, g0, x, n0, n, k, h.kT, soft, e1, e2, s1, Z, sv);
        gap = (e2 - e1 < 1e-9) ? 1 : 0;
#pragma unroll
        for (int i = 0; i < NM; ++i)
            if (i < n) nout[i] = n0[i] + (int)(s1 >> i & 1u);
        if (nbout) {
#pragma unroll
            for (int i = 0; i < NM; ++i)
                if (i < n)
                    nbout[i] = soft ? (double)n0[i] + sv[i] / Z
                                    : (double)(n0[i] + (int)(s1 >> i & 1u));
        }
        return closed ? closed_states(n, k) : (int64_t)1 << n;
    }
    // any other set: argmin and runner-up with the y = A 1_s walk
    const int m = __popc(fm);
    const uint64_t pos = free_positions(fm);
    const int steps = 1 << m;
    double y[NM];
    double e1 = INFINITY, e2 = INFINITY;
    uint32_t s1 = 0;
    int64_t scored = 0;
    {
        uint32_t s = 0;
        int pc = 0;
        walk_start<NM>(L.A, s, y);
        for (int step = 0; step < steps; ++step) {
            if (step) walk_flip<NM>(L.A, pos, step, s, pc, y);
            if (k < 0 || pc == k) {
                const double e = walk_energy<NM>(g0, y, u0, s);
                ++scored;
                if (better(e, s, e1, s1)) { e2 = e1; e1 = e; s1 = s; }
                else if (e < e2) e2 = e;
            }
        }
    }
    gap = (e2 - e1 < 1e-9) ? 1 : 0;
#pragma unroll
    for (int i = 0; i < NM; ++i)
        if (i < n) nout[i] = n0[i] + (int)(s1 >> i & 1u);
    if (nbout) {
        const double kT = h.kT;
        if (kT > 0.0) {
            double Z = 0.0, sv[NM];
#pragma unroll
            for (int i = 0; i < NM; ++i) sv[i] = 0.0;
            uint32_t s = 0;
            int pc = 0;
            walk_start<NM>(L.A, s, y);
            for (int step = 0; step < steps; ++step) {
                if (step) walk_flip<NM>(L.A, pos, step, s, pc, y);
                if (k < 0 || pc == k) {
                    const double w = exp(-(walk_energy<NM>(g0, y, u0, s) - e1) / kT);
                    Z += w;
#pragma unroll
                    for (int i = 0; i < NM; ++i)
                        if (s >> i & 1u) sv[i] += w;
                }
            }
#pragma unroll
            for (int i = 0; i < NM; ++i)
                if (i < n) nbout[i] = (double)n0[i] + sv[i] / Z;
        } else {
#pragma unroll
            for (int i = 0; i < NM; ++i)
                if (i < n) nbout[i] = (double)(n0[i] + (int)(s1 >> i & 1u));
        }
    }
    return scored;
}

// One block of one wave per work item, largest dot counts first, handed out by
// the hardware as waves end.  What bounds it is the FP64 instructions of a lane's
// chain and, beside them, the latency of the reads before it: the item's diagram,
// its header, then the tables and the voltages.  512 diagrams of 2..8 dots, 64 x 64
// pixels: 438 -> 202 us a call, of which
//     the walk's blocks left out by their bound                  438 -> 365 us,
//     tables in LDS rather than scalar loads                      -> 316 us,
//     this order rather than persistent waves with a queue of
//     sharded cursors (a wave that had claimed its next item
//     could still be at a long one when the others had ended)     -> 250 us,
//     a QP of one form and no masks, nothing spilled (qp_solve)   -> 202 us.
// With a new plan at every call (one upload, C_dd of the prologue kept in LDS) a call
// takes 223 us.  Three waves per SIMD (163 registers); two take as long, four 216 us.
// Reading voltages and writing results through LDS, row by row, was slower (287 for
// 250).
template <int NM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NM <= 8 ? 3 : 1))) void k_batch(
    const BatchHdr *__restrict__ hdr, const DiagRec *__restrict__ recs,
    const double *__restrict__ mats, const int32_t *__restrict__ owner,
    int64_t item0, const double *__restrict__ V, int32_t *__restrict__ n_out,
    double *__restrict__ nbar, int64_t *__restrict__ counters)
{
    __shared__ DiagLds<NM> L;
    const int lane = threadIdx.x;
    const int64_t item = item0 + blockIdx.x;
    const int d = __builtin_amdgcn_readfirstlane(owner[item]);
    const BatchHdr h = hdr[d];
    const DiagRec *dr = recs + d;
    const double one_c = dr->one_c;
#pragma unroll
    for (int r = 0; r < NM * kMaxDot / 64; ++r) {
        const int e = r * 64 + lane;
        L.A[e] = dr->A[e];
        L.K[e] = h.closed ? dr->Cdd[e] - dr->c[e / kMaxDot] * dr->c[e % kMaxDot] / one_c
                          : dr->Cdd[e];
    }
#pragma unroll
    for (int r = 0; r < NM * kMaxGate / 64; ++r) {
        const int e = r * 64 + lane;
        L.Cgt[(e % kMaxGate) * NM + e / kMaxGate] = dr->Cgd[e];
    }
    if (lane < NM) L.c[lane] = dr->c[lane];
    if (NM <= 8) {
#pragma unroll
        for (int r = 0; r < 4; ++r) L.hs[r * 64 + lane] = dr->hs[r * 64 + lane];
        __syncthreads();
        const int hi = lane & ~3, i = lane & 3;
        L.bb.hd[lane >> 2][i] = L.hs[4 * hi + (1 << i)] - L.hs[4 * hi];
        double neg = 0.0;
#pragma unroll
        for (int r = 1; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < r; ++q) neg += fmax(0.0, -L.A[r * kMaxDot + q]);
        const int x = lane >> 3, y = lane & 7;
        const double hm = wave_sum(x < NM && y < NM ? fabs(L.A[x * kMaxDot + y]) : 0.0);
        if (lane == 0) {
            L.bb.neg = neg;
            L.bb.hmax = 0.5 * hm;
        }
    }
    __syncthreads();
    const int64_t p = (item - h.tile0) * 64 + lane;
    const bool on = p < h.P;
    // x_u = C_gd V, gate by gate: each voltage is read, or formed from
    // the diagram's sweep, once, and every x_u,i still sums over j in
    // increasing order
    double xu[NM];
#pragma unroll
    for (int i = 0; i < NM; ++i) xu[i] = 0.0;
    auto add_gate = [&](int j, double vj) {
#pragma unroll
        for (int i = 0; i < NM; ++i)
            xu[i] += L.Cgt[j * NM + i] * vj;  // (0 past the last dot)
    };
    if (h.nx > 0) {
        const double *gv = mats + h.grid_off;
        const double *sc = gv + 3 * h.g;  // a0, da, a1, b0, db, b1
        const uint32_t nx = (uint32_t)h.nx, row = (uint32_t)p / nx;
        const double va =
            lin_point((int32_t)((uint32_t)p - row * nx), (int32_t)nx, sc[0], sc[1], sc[2]);
        const double vb = lin_point((int32_t)row, (int32_t)h.ny, sc[3], sc[4], sc[5]);
        for (int j = 0; j < h.g; ++j)
            add_gate(j, sweep_volt(gv[j], gv[h.g + j], gv[2 * h.g + j], va, vb));
    } else {
        const double *Vp = V + h.v_off + p * h.g;
        for (int j = 0; j < h.g; ++j) add_gate(j, on ? Vp[j] : 0.0);
    }
    int qp = 0, fail = 0, dbl = 0, gap = 0;
    int64_t cand = 0;
    if (on)
        cand = batch_pixel<NM>(L, h, one_c, xu, n_out + h.out_off + p * h.n,
                               nbar ? nbar + h.out_off + p * h.n : nullptr, qp, fail, dbl, gap);
    const auto count = [&](int which, bool b) {
        const int64_t c = __popcll(__ballot(b));
        if (lane == 0) block_add_counter(counters, which, c);
    };
    count(C_PIXELS, on);
    count(C_QP, qp != 0);
    count(C_QP_FAIL, fail != 0);
    count(C_DOUBLED, dbl != 0);
    count(C_GAP_1E9, gap != 0);
    cand = (int64_t)wave_sum((double)cand);
    if (lane == 0) block_add_counter(counters, C_CANDIDATES, cand);
}

hipError_t launch_batch(const BatchHdr *hdr, const DiagRec *recs, const double *mats,
                        const int32_t *owner, int64_t tiles, const double *V, int32_t *n_out,
                        double *nbar, int64_t *counters, int max_dot, hipStream_t s)
{
    if (tiles < 1) return hipErrorInvalidValue;
    // (a launch holds fewer than 2^32 threads)
    constexpr int64_t kMostItems = (int64_t)1 << 25;
    const auto go = [&](auto kernel) {
        for (int64_t item0 = 0; item0 < tiles; item0 += kMostItems) {
            const int64_t items = tiles - item0 < kMostItems ? tiles - item0 : kMostItems;
            hipLaunchKernelGGL(kernel, dim3((unsigned)items), dim3(64), 0, s, hdr, recs, mats,
                               owner, item0, V, n_out, nbar, counters);
            if (const hipError_t e = hipGetLastError()) return e;
        }
        return hipSuccess;
    };
    return max_dot <= 4 ? go(k_batch<4>) : max_dot <= 8 ? go(k_batch<8>) : go(k_batch<16>);
}

}  // namespace qa
