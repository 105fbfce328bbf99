// qa_sensor.hip -- charge-sensor response (Sec. 5.1) after the array's
// charges are known.
//
// The problem's last S dots are sensor dots.  The array dots' charges n_a
// come from the array's own ground state or softargmin (computed with the
// array block of C_dd and C_gd: the sensors left out, every gate's
// cross-talk kept).  With n_a fixed, each pixel's sensor charges minimise
// U(n) = 1/2 (n - x_u)^T A (n - x_u), A = C_dd^{-1} of the whole system, over
// the floor/ceil box around the sensors' continuous minimum (clipped at 0:
// one sensor is then exact, a 1-D convex quadratic); the sensor potentials
// are v = A (n - x_u) (Eq. for the potential).  Adding a carrier to sensor s
// costs v_s + A_ss/2, removing one -v_s + A_ss/2; the response is the peak
// profile (Lorentzian or Gaussian, width gamma) of each, summed (the removal
// term only for an occupied sensor), so it peaks at the Coulomb-peak
// conditions on either side.  Noise on top, from draws passed in:
// white (amplitude x a standard-normal draw per sample), 1/f (Voss-McCartney:
// K octave sources, source k redrawn every 2^k samples, summed over sqrt K)
// and random telegraph jumps (the state flips where a uniform draw falls
// below the rate; amplitude x state), samples in pixel order.
#include "qa_device.h"

namespace qa {

constexpr int kMaxSensor = 4;

// A block's share of the samples, in pixel order: tiles of kSensorTile pixels, a
// pixel per thread of waves 1..3, from `first` on.
constexpr int kSensorWaves = 3;
constexpr int kSensorThreads = (1 + kSensorWaves) * kWave;
constexpr int kSensorTile = kSensorWaves * kWave;
constexpr int kSensorBlocks = 1024;
static_assert(kSensorBlocks == kSensorParities, "a parity word per block");

// the parity of the flips (uniform draw below the rate) in every block's share of
// k_sensor, bit s: sensor s
__global__ __launch_bounds__(kSensorThreads) void k_flip_parity(int64_t P, int n_sensor,
                                                                int64_t share,
                                                                const double *__restrict__ u,
                                                                double rate,
                                                                int32_t *__restrict__ parity)
{
    __shared__ uint32_t sw[kSensorThreads / kWave];
    const int64_t first = (int64_t)blockIdx.x * share;
    const int64_t last = first + share < P ? first + share : P;
    uint32_t acc = 0;
    for (int64_t t = first + threadIdx.x; t < last; t += kSensorThreads)
        for (int s = 0; s < n_sensor; ++s) acc ^= u[t * n_sensor + s] < rate ? 1u << s : 0u;
    uint32_t bits = 0;
    for (int s = 0; s < n_sensor; ++s)
        bits |= (uint32_t)(__popcll(__ballot(acc >> s & 1u)) & 1) << s;
    if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = bits;
    __syncthreads();
    if (threadIdx.x == 0) parity[blockIdx.x] = (int32_t)(sw[0] ^ sw[1] ^ sw[2] ^ sw[3]);
}

struct SensorArgs {
    int shape, octaves;
    double gamma, white, pink, jump, rate;
    const double *V;
    int64_t P, share;  // share: pixels of a block
    const int32_t *n_int;
    const double *n_dbl;
    const double *white_draws, *pink_draws, *jump_draws;
    const int32_t *parity;  // of the blocks' flips (jump_draws given)
    double *signal;
};

// Bound by latency at the usual sizes: wave 0 inverts C_dd (3 us) while the pixel
// waves read what they need of their first tile and form x_u; one barrier hands A
// over.  The telegraph state before a tile is the parity of the flips before it:
// the shares' parities (k_flip_parity), then the tiles' own, by wave ballots.
// 8 dots and a sensor, 10^4 pixels: 12.4 us with the inverse ahead of all reads and
// another 12.1 us for a pass over the samples by one block for the telegraph noise
// (which grew with the samples); now 7.0 us and 2.4 us for the shares' parities.
// NA: array dots, 8 or 16.
template <int S, int NA, bool ARGS>
__global__ __launch_bounds__(kSensorThreads) void k_sensor(
    const DiagRec *__restrict__ dr, const SensorArgs a,
    const std::conditional_t<ARGS, SetupIn, int> in)
{
    __shared__ double sA[kMaxDot * kMaxDot];
    __shared__ double red[8];
    __shared__ double sG[kMaxGate * kMaxDot];  // C_gd transposed: sG[j * kMaxDot + i]
    __shared__ double sB[S * S];               // (A_ss)^{-1}
    __shared__ uint32_t sflip[2][kSensorWaves], sbefore;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int n, g;
    if constexpr (ARGS) {
        n = in.n, g = in.g;
    } else {
        n = dr->n, g = dr->g;
    }
    const int Na = n - S, tri = n * (n + 1) / 2;
    double m4[4], gv[2];
    {
        // (entries past n or g: the first one read again, then replaced)
        const int j = tid & 15, b = (tid >> 4) & 3;
        if (wave == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * b + q, hi = i > j ? i : j, lo = i > j ? j : i;
                if constexpr (ARGS) m4[q] = in.v[hi < n ? hi * (hi + 1) / 2 + lo : 0];
                else m4[q] = dr->Cdd[i * kMaxDot + j];
            }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int e = r * kSensorThreads + tid, jj = e / kMaxDot, i = e % kMaxDot;
            if constexpr (ARGS) gv[r] = in.v[i < n && jj < g ? tri + i * g + jj : 0];
            else gv[r] = dr->Cgd[i * kMaxGate + jj];
        }
        if (wave == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * b + q;
                m4[q] = i < n && j < n ? m4[q] : (i == j ? 1.0 : 0.0);
            }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int e = r * kSensorThreads + tid, jj = e / kMaxDot, i = e % kMaxDot;
            sG[e] = i < n && jj < g ? gv[r] : 0.0;
        }
    }
    __syncthreads();
    const int64_t P = a.P;
    const int64_t first = (int64_t)blockIdx.x * a.share;
    const int64_t last = first + a.share < P ? first + a.share : P;
    uint32_t state = 0;  // bit s: sensor s is up after the samples so far
    for (int64_t t0 = first; t0 < last; t0 += kSensorTile) {
        const int64_t p = t0 + (tid - kWave);
        const bool on = wave > 0 && p < last;
        const int64_t pc = on ? p : first;
        double xu[NA], xs[S], w[S], up[S], na[NA], pink[S];
        if (wave > 0) {
            // Every read of the pixel is issued before the first is used.  (Past the
            // last dot, gate or octave the last or first one is read again: a
            // condition would put a branch and a wait at each.)
            double v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = a.V[pc * g + (j < g ? j : g - 1)];
            int32_t ni[NA] = {};
#pragma unroll
            for (int i = 0; i < NA; ++i) na[i] = 0.0;
            if (Na && a.n_int) {
#pragma unroll
                for (int i = 0; i < NA; ++i) ni[i] = a.n_int[pc * Na + (i < Na ? i : 0)];
            } else if (Na) {
#pragma unroll
                for (int i = 0; i < NA; ++i) na[i] = a.n_dbl[pc * Na + (i < Na ? i : 0)];
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                w[s] = a.white_draws ? a.white_draws[pc * S + s] : 0.0;
                up[s] = a.jump_draws ? a.jump_draws[pc * S + s] : 0.0;
            }
            if (a.pink_draws) {
                // octave k of sensor s starts after the earlier sources' draws
                int64_t off = 0;
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    pink[s] = 0.0;
                    for (int k0 = 0; k0 < a.octaves; k0 += 8) {
                        double y[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) {
                            const int kk = k0 + k < a.octaves ? k0 + k : 0;
                            y[k] = a.pink_draws[k0 + k < a.octaves ? off + (pc >> kk) : 0];
                            if (k0 + k < a.octaves) off += (P + ((int64_t)1 << kk) - 1) >> kk;
                        }
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            if (k0 + k < a.octaves) pink[s] += y[k];
                    }
                }
            }
            if (a.n_int) {
#pragma unroll
                for (int i = 0; i < NA; ++i) na[i] = (double)ni[i];
            }
            // x_u = C_gd V of every dot (xs: of the sensors), eight gates a time
#pragma unroll
            for (int i = 0; i < NA; ++i) xu[i] = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) xs[s] = 0.0;
            for (int j0 = 0; j0 < g; j0 += 8) {
                if (j0)
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        v[j] = a.V[pc * g + (j0 + j < g ? j0 + j : g - 1)];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (j0 + j >= g) break;
                    const double *row = sG + (j0 + j) * kMaxDot;
#pragma unroll
                    for (int i = 0; i < NA; ++i) xu[i] += row[i] * v[j];
#pragma unroll
                    for (int s = 0; s < S; ++s) xs[s] += row[Na + s] * v[j];
                }
            }
            if (a.jump_draws) {
                uint32_t bits = 0;
#pragma unroll
                for (int s = 0; s < S; ++s)
                    bits |= (uint32_t)(__popcll(__ballot(on && up[s] < a.rate)) & 1) << s;
                if (lane == 0) sflip[(t0 - first) / kSensorTile & 1][wave - 1] = bits;
                if (wave == 1 && t0 == first) {
                    // the shares before this one
                    uint32_t acc = 0;
                    for (int k = lane; k < (int)blockIdx.x; k += kWave) acc ^= (uint32_t)a.parity[k];
                    uint32_t before = 0;
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        before |= (uint32_t)(__popcll(__ballot(acc >> s & 1u)) & 1) << s;
                    if (lane == 0) sbefore = before;
                }
            }
        } else if (t0 == first) {
            __builtin_amdgcn_s_setprio(3);
            prep_inverse_wave(m4, n, sA, red);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // inverse of the sensor block of A by Gauss-Jordan (positive
            // definite, no pivoting), in every lane
            double m[S][2 * S];
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int j = 0; j < 2 * S; ++j)
                    m[i][j] = (j < S) ? sA[(Na + i) * kMaxDot + Na + j] : (j - S == i ? 1.0 : 0.0);
#pragma unroll
            for (int k = 0; k < S; ++k) {
                const double r = 1.0 / m[k][k];
#pragma unroll
                for (int j = 0; j < 2 * S; ++j) m[k][j] *= r;
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    if (i == k) continue;
                    const double f = m[i][k];
#pragma unroll
                    for (int j = 0; j < 2 * S; ++j) m[i][j] -= f * m[k][j];
                }
            }
            if (lane == 0)
#pragma unroll
                for (int i = 0; i < S; ++i)
#pragma unroll
                    for (int j = 0; j < S; ++j) sB[i * S + j] = m[i][S + j];
            __builtin_amdgcn_s_setprio(0);
        }
        __syncthreads();
        if (wave > 0) {
            const double *As = sA + Na * kMaxDot;  // the sensors' rows of A
            double white[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                white[s] = w[s];
                w[s] = 0.0;
            }
            // w = A_sa (n_a - x_u,a): the array's pull on each sensor
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (i < Na) {
                    const double za = na[i] - xu[i];
#pragma unroll
                    for (int s = 0; s < S; ++s) w[s] += As[s * kMaxDot + i] * za;
                }
            // continuous minimum over the sensor charges and its box
            int base[S];
            double ss[S][S];  // A_ss
#pragma unroll
            for (int s = 0; s < S; ++s) {
                double x = xs[s];
#pragma unroll
                for (int r = 0; r < S; ++r) {
                    x -= sB[s * S + r] * w[r];
                    ss[s][r] = As[s * kMaxDot + Na + r];
                }
                base[s] = (int)floor(fmax(x, 0.0));
            }
            // the sensor-dependent part of U: d^T w + 1/2 d^T A_ss d, d = n_s - x_u,s;
            // ties to the lexicographically smallest charges (sensor 0 most
            // significant): candidates in that order, strict improvement only
            double best = INFINITY;
            int bits = 0;
            for (int c = 0; c < (1 << S); ++c) {
                double d[S], e = 0.0;
#pragma unroll
                for (int s = 0; s < S; ++s)
                    d[s] = (double)(base[s] + ((c >> (S - 1 - s)) & 1)) - xs[s];
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    double q = 0.0;
#pragma unroll
                    for (int r = 0; r < S; ++r) q += ss[s][r] * d[r];
                    e += d[s] * (w[s] + 0.5 * q);
                }
                if (e < best) { best = e; bits = c; }
            }
            uint32_t before = 0;
            if (a.jump_draws) {
                if (t0 == first) state = sbefore;
                before = state;
#pragma unroll
                for (int k = 0; k < kSensorWaves; ++k) {
                    const uint32_t f = sflip[(t0 - first) / kSensorTile & 1][k];
                    state ^= f;
                    if (k < wave - 1) before ^= f;
                }
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int ns = base[s] + ((bits >> (S - 1 - s)) & 1);
                // sensor potential v_s = w_s + (A_ss d)_s
                double vs = w[s];
#pragma unroll
                for (int r = 0; r < S; ++r) {
                    const double d = (double)(base[r] + ((bits >> (S - 1 - r)) & 1)) - xs[r];
                    vs += ss[s][r] * d;
                }
                const double half = 0.5 * ss[s][s];
                const double xp = (vs + half) / a.gamma, xm = (-vs + half) / a.gamma;
                double r;
                if (a.shape == 0) {
                    r = 1.0 / (1.0 + xp * xp) + (ns > 0 ? 1.0 / (1.0 + xm * xm) : 0.0);
                } else {
                    r = exp(-0.5 * xp * xp) + (ns > 0 ? exp(-0.5 * xm * xm) : 0.0);
                }
                if (a.white_draws) r += a.white * white[s];
                if (a.pink_draws) r += a.pink * pink[s] / sqrt((double)a.octaves);
                if (a.jump_draws) {
                    const unsigned long long f = __ballot(on && up[s] < a.rate);
                    const int incl = __popcll(f & (~0ull >> (63 - lane)));  // flips up to this lane
                    if ((incl + (int)(before >> s & 1u)) & 1) r += a.jump;
                }
                if (on) a.signal[p * S + s] = r;
            }
        }
    }
}

hipError_t launch_sensor(const DiagRec *dr, const SetupIn *in, int n_dot, int n_sensor, int shape,
                         double gamma, const double *V, int64_t P, const int32_t *n_int,
                         const double *n_dbl, const double *white_draws, double white,
                         const double *pink_draws, double pink, int octaves,
                         const double *jump_draws, double jump, double rate, int32_t *parity,
                         double *signal, hipStream_t s)
{
    if (P <= 0) return hipSuccess;
    if (n_sensor < 1 || n_sensor > kMaxSensor) return hipErrorInvalidValue;
    const int64_t tiles = (P + kSensorTile - 1) / kSensorTile;
    const int64_t per = (tiles + kSensorBlocks - 1) / kSensorBlocks;
    const int64_t share = per * kSensorTile;
    const dim3 grid((unsigned)((P + share - 1) / share));
    if (jump_draws) {
        // (the last share's flips come before no other)
        if (grid.x > 1)
            hipLaunchKernelGGL(k_flip_parity, dim3(grid.x - 1), dim3(kSensorThreads), 0, s, P,
                               n_sensor, share, jump_draws, rate, parity);
    }
    const SensorArgs a{shape,   octaves, gamma,       white,      pink,       jump,   rate,  V,
                       P,       share,   n_int,       n_dbl,      white_draws, pink_draws,
                       jump_draws, parity, signal};
    const auto go = [&](auto kernel, const auto &src) {
        hipLaunchKernelGGL(kernel, grid, dim3(kSensorThreads), 0, s, dr, a, src);
    };
    const auto with = [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if (n_dot - S <= 8 && in) go(k_sensor<S, 8, true>, *in);
        else if (n_dot - S <= 8) go(k_sensor<S, 8, false>, 0);
        else if (in) go(k_sensor<S, 16, true>, *in);
        else go(k_sensor<S, 16, false>, 0);
    };
    switch (n_sensor) {
    case 1: with(std::integral_constant<int, 1>{}); break;
    case 2: with(std::integral_constant<int, 2>{}); break;
    case 3: with(std::integral_constant<int, 3>{}); break;
    default: with(std::integral_constant<int, 4>{}); break;
    }
    return hipGetLastError();
}

}  // namespace qa
