// Single-wave and whole-workgroup helpers of the small FP64 algebra: LDS
// matrix moves, fixed-order sums of per-workgroup partials, a Cholesky
// factorisation with inverse, and a one-sided Jacobi SVD run by two waves.
// Shared by the panel kernels of the loop and of the relaxed iteration.
#pragma once

#include "launch.hpp"

namespace rpca {
namespace {

constexpr double JACOBI_EPS = 1e-15;
// Pairs with |a_p . a_q| <= JACOBI_ABS ||M||_F^2 are left alone: such a coupling
// moves the leading singular vectors by about that relative amount, and the
// trailing (negligible) columns would otherwise keep rotating on rounding noise.
constexpr double JACOBI_ABS = 1e-17;
constexpr int JACOBI_MAX_SWEEPS = 40;
// Cyclic Jacobi converges quadratically: once every rotation of a sweep was by
// an angle below JACOBI_QUAD (the angle is the coupling over the gap of the
// pair), the angles a further sweep would take are of the order
// JACOBI_QUAD^2, and the confirming sweep is skipped.
constexpr double JACOBI_QUAD = 1e-8;
// The same for M formed from FP32 products: the angles a further sweep would
// take (about 4e-8) are below the rounding of those products (6e-8) and of the
// FP32 factors the result is stored in, and below the initial subspace
// iteration's FP32 tolerance (3e-6), so stopping here changes nothing the FP32
// path can resolve. It saves about one sweep of the tail per body.
constexpr double JACOBI_QUAD_F32 = 2e-4;
constexpr double CHOL_DEAD_REL = 1e-26;

// ---- single-wave helpers (the last workgroup's tail) ---------------------------

__device__ inline int lane_id() { return threadIdx.x & (WAVE - 1); }
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int K>
__device__ inline void w_store(const double* s, double* __restrict__ g) {
    for (int e = lane_id(); e < K * K; e += WAVE) g[(e / K) * KMAX + (e % K)] = s[e];
    wave_sync();
}
// Sums of the per-workgroup partials of a kernel whose first gU workgroups
// cover the U side (rows of m) and the next gV the V side (rows of n). Job j
// sums entry e < E of the partial at offset (j / 2) * KMAX^2 of every
// workgroup of side j % 2, into out[j * E + e].
// The whole workgroup (NT threads) takes part. Thread t takes pair
// q = t % PAIRS (job q / E, entry q % E) and split s = t / PAIRS and sums the
// partials b = s, s + S, ... in order; the S split sums of a pair are then
// added in order of s. Up to L loads per thread are in flight at once, so a
// round over up to L S partials costs one memory latency. part: NT doubles
// of LDS.
// SYM > 0: jobs 2 and up are symmetric SYM x SYM matrices of which only the
// entries on and above the diagonal are there (and are summed).
template <int E, int J, int NT, int L = 16, int SYM = 0>
__device__ __forceinline__ void block_sum_partials(const double* __restrict__ gpart, int gU, int gV, double* out, double* part) {
    constexpr int PAIRS = J * E;
    constexpr int PR = PAIRS >= NT ? NT : PAIRS;   // pairs per round
    constexpr int S = NT / PR;                     // splits per pair
    // L: loads in flight per thread
    const int t = threadIdx.x;
    for (int q0 = 0; q0 < PAIRS; q0 += PR) {
        const int sp = t / PR, q = q0 + t % PR;
        double acc = 0.0;
        const int j = q / E, e = q - (q / E) * E;
        if (sp < S && q < PAIRS && !(SYM > 0 && j >= 2 && e / (SYM > 0 ? SYM : 1) > e % (SYM > 0 ? SYM : 1))) {
            const int first = (j & 1) ? gU : 0, count = (j & 1) ? gV : gU;
            const double* g = gpart + (size_t)first * GPART_STRIDE + (j >> 1) * (KMAX * KMAX) + e;
            for (int b0 = sp; b0 < count; b0 += L * S) {
                double v[L];
#pragma unroll
                for (int u = 0; u < L; ++u) {
                    const int b = b0 + u * S;
                    v[u] = b < count ? g[(size_t)b * GPART_STRIDE] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < L; ++u) acc += v[u];
            }
        }
        if (t < S * PR) part[t] = acc;
        __syncthreads();
        if (t < PR && q0 + t < PAIRS) {
            double v = 0.0;
            for (int u = 0; u < S; ++u) v += part[u * PR + t];
            out[q0 + t] = v;
        }
        __syncthreads();
    }
}

template <int CTRL> __device__ inline double dpp64(double x);
__device__ inline double row16_sum(double x);
__device__ inline double row16_max(double x);
__device__ inline double readlane64(double x, int l);

// Sum of the per-tile residuals (and, if want_max, the max of the per-tile
// max |D_ij| stored after them) by the whole workgroup, in a fixed order.
// out[0] = sum, out[1] = max. part: at least 2 * NT / 16 doubles of LDS.
// Split in two: block_resid_fetch issues the loads of the first RESID_LD * NT
// tiles into registers (so that other loads can follow before they are
// used), block_resid adds them, and any further tiles, in tile order per thread.
constexpr int RESID_LD = 2;
template <int NT>
__device__ inline void block_resid_fetch(const double* __restrict__ resid, int n_tiles, bool want_max,
                                         double (&v)[RESID_LD], double (&w)[RESID_LD]) {
#pragma unroll
    for (int u = 0; u < RESID_LD; ++u) {
        const int b = threadIdx.x + u * NT;
        v[u] = b < n_tiles ? resid[b] : 0.0;
        w[u] = (want_max && b < n_tiles) ? resid[n_tiles + b] : 0.0;
    }
}
template <int NT>
__device__ __forceinline__ void block_resid(const double* __restrict__ resid, int n_tiles, bool want_max,
                            const double (&v)[RESID_LD], const double (&w)[RESID_LD], double* part, double* out) {
    const int t = threadIdx.x;
    double sm = 0.0, mx = 0.0;
#pragma unroll
    for (int u = 0; u < RESID_LD; ++u) {
        sm += v[u];
        mx = fmax(mx, w[u]);
    }
    for (int b = t + RESID_LD * NT; b < n_tiles; b += NT) {
        sm += resid[b];
        if (want_max) mx = fmax(mx, resid[n_tiles + b]);
    }
    // sums and maxima over each row of 16 lanes by DPP; the four rows of a
    // wave go to LDS separately
    sm = row16_sum(sm);
    mx = row16_max(mx);
    constexpr int NW = NT / 16;
    static_assert(NW <= WAVE, "one row sum per lane of the first wave");
    if ((t & 15) == 0) {
        part[t / 16] = sm;
        part[NW + t / 16] = mx;
    }
    __syncthreads();
    if (t < WAVE) {
        double a = t < NW ? part[t] : 0.0, m = t < NW ? part[NW + t] : 0.0;
        a = row16_sum(a);
        m = row16_max(m);
        a = (readlane64(a, 0) + readlane64(a, 16)) + (readlane64(a, 32) + readlane64(a, 48));
        m = fmax(fmax(readlane64(m, 0), readlane64(m, 16)), fmax(readlane64(m, 32), readlane64(m, 48)));
        if (t == 0) {
            out[0] = a;
            out[1] = m;
        }
    }
    __syncthreads();
}

__device__ inline double readlane64(double x, int l) {
    const int64_t u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Cholesky factor and its inverse of a K x K matrix G = R^T R (all K x K, ld K,
// LDS; R upper triangular) by the lanes c of a group of a wave: lane c < K owns
// column c of G, lane K + c column c of the identity, in registers. Step j
// leaves row j of R in the first, row j of R^{-T} in the second (forward
// elimination of [G | I]), so the inverse needs no pass of its own. Row j of the
// reduced matrix is handed round through LDS (buf, K values): one write and one
// read per step instead of a broadcast by lane per entry (two at K = 11: 7.4 ->
// 3.6 us). A pivot that vanishes (d <= CHOL_DEAD_REL * G_jj, or G_jj ~ 0) marks a
// numerically dependent column: its row of R and column of R^{-1} are 0.
template <int K>
__device__ __forceinline__ void chol_group(const double* G, double* R, double* Ri, double* buf, int c) {
    double a[K];
#pragma unroll
    for (int i = 0; i < K; ++i) a[i] = c < K ? G[i * K + c] : (c - K == i ? 1.0 : 0.0);
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (c < K) buf[c] = a[j];
        const double gjj = G[j * K + j];
        wave_sync();
        double v[K];
#pragma unroll
        for (int i = j; i < K; ++i) v[i] = buf[i];
        wave_sync();
        const double d = v[j];
        const bool live = gjj > 1e-300 && d > CHOL_DEAD_REL * gjj;
        const double iv = live ? rsqrt(d) : 0.0;   // one reciprocal square root, no division
        const double r = c < j ? 0.0 : a[j] * iv;
        if (c < K) R[j * K + c] = r;
        else if (c < 2 * K) Ri[(c - K) * K + j] = a[j] * iv;
#pragma unroll
        for (int i = j + 1; i < K; ++i) a[i] = fma(-(v[i] * iv), a[j] * iv, a[i]);
    }
}

// Two such factorisations by one wave (K <= 16: 2K lanes each)
template <int K>
__device__ __forceinline__ void w_chol_inv2(const double* G0, double* R0, double* Ri0, const double* G1, double* R1,
                                            double* Ri1) {
    static_assert(K <= 16, "2K lanes of a half wave per matrix");
    __shared__ double buf[2][KMAX];
    const int lane = lane_id(), h = lane >> 5;
    chol_group<K>(h ? G1 : G0, h ? R1 : R0, h ? Ri1 : Ri0, buf[h], lane & 31);
    wave_sync();
}

template <int CTRL> __device__ inline double dpp64(double x) {
    const int64_t u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
__device__ inline double row16_sum(double x) {
    x += dpp64<0xB1>(x);
    x += dpp64<0x4E>(x);
    x += dpp64<0x141>(x);
    x += dpp64<0x128>(x);
    return x;
}
__device__ inline double row16_max(double x) {
    x = fmax(x, dpp64<0xB1>(x));
    x = fmax(x, dpp64<0x4E>(x));
    x = fmax(x, dpp64<0x141>(x));
    x = fmax(x, dpp64<0x128>(x));
    return x;
}
// Sum over aligned groups of LP lanes (LP = 1, 2, 4, 8, 16), result in every lane.
template <int LP> __device__ inline double group_sum(double x) {
    if constexpr (LP >= 2) x += dpp64<0xB1>(x);    // quad_perm[1,0,3,2]: lane ^ 1
    if constexpr (LP >= 4) x += dpp64<0x4E>(x);    // quad_perm[2,3,0,1]: lane ^ 2
    if constexpr (LP >= 8) x += dpp64<0x141>(x);   // row_half_mirror:    lane ^ 7
    if constexpr (LP >= 16) x += dpp64<0x128>(x);  // row_ror:8:          lane ^ 8
    return x;
}

constexpr int pow2_floor(int x) { int p = 1; while (p * 2 <= x) p *= 2; return p; }

// ---- one-sided (Hestenes) Jacobi SVD of a small matrix -------------------------
//
// A (N x N, LDS, column-major) in the registers of one wave: the N / 2 disjoint
// column pairs of a round-robin round are processed at once. A pair is rotated
// when |a_p . a_q| > JACOBI_EPS ||a_p|| ||a_q|| and above the absolute floor
// JACOBI_ABS ||A||_F^2 (pairs of negligible columns would otherwise rotate on
// rounding noise), unless both columns have ||a||^2 <= neg2 ||A||_F^2 (columns the
// caller discards: a rotation never raises the smaller norm of a pair). Sweeps
// stop when no pair was rotated, or (QUAD_STOP) after a sweep whose rotation
// angles were all below quad (default JACOBI_QUAD); callers that difference
// the result keep the confirming sweep.
//
// Bound by one wave's instruction stream: a round is a serial chain (an inner
// product, a rotation, the columns handed to the next round's pairs) and a
// sweep N - 1 of them. So everything off that chain is kept off it:
//   - Lane l holds rows l / PL + NSUB u of the pair l % PL: handing the columns
//     on is a move by one lane (DPP), inner products are sums over the upper
//     lane bits (DPP, v_permlane swaps), and LDS is only written.
//   - The right vectors, which no round reads, are rotated by a second wave from
//     the cosines and sines left in LDS, one sweep behind (two buffers, one
//     barrier per sweep).
//   - Squared norms travel with their columns and are formed anew each sweep: a
//     rotation changes them by +- tan(theta) (a_p . a_q). Within a sweep they are
//     off by a few roundings of the largest column's square (about 1e-16 ||A||_F^2,
//     more than the absolute floor), so a small column's angle can be wrong there;
//     the next sweep starts from norms formed anew.
//   - The angle is found in FP32 (A is scaled by a power of two to a norm near
//     1), tan(theta) good to about 2^-22, and refined by one Newton step in FP64,
//     good to about 2^-44; cosine and sine are formed from it in FP64. Without
//     that step a rotation leaves 2^-22 of its coupling phi sigma_i^2, which after a
//     last sweep with angles phi near 1e-8 is 2^-22 phi sigma_i / sigma_j between the left
//     vectors: orthogonality 1e-13 at sigma_i / sigma_j = 100, 1e-11 at 10^4.
// With the columns in LDS, both matrices in one wave and FP64 angles a round took
// 0.36 us at N = 12 and 0.55 at N = 22; now 0.24 and 0.33 (gather of the
// initialisation at m = n = 10^4, 2K = 12: 39 -> 30 us; at 2 10^4, 2K = 22: 115 ->
// 90 us; FP64 complement at n = 1000, 2K = 12: 32 -> 24 us). The Newton step's part of
// such a launch is about 2 %: 26.8 -> 27.4 us, 89.1 -> 89.6 and 22.1 -> 23.6.
//
// jacobi_svd is called by every live wave of the workgroup with its index: wave 0
// works on A, wave 1 on the right vectors, others only take part in the
// barriers. On return (after a barrier) sig[] is descending and Uo / Vo hold
// the left / right singular vectors as columns (column-major). Wave 0 returns the
// sweep count. A is unchanged.
template <int N> struct JacobiGeom {
    static_assert(N % 2 == 0 && N <= 2 * KMAX, "even N up to 2*KMAX");
    static constexpr int P = N / 2;                 // pairs
    static constexpr int PL = P <= 8 ? 8 : 16;      // lanes per group of pairs
    static constexpr int NSUB = WAVE / PL;          // lanes per pair
    static constexpr int E = (N + NSUB - 1) / NSUB; // rows of a column per lane
};
enum JacobiFlag : int { JACOBI_GO = 0, JACOBI_LAST = 1 };
template <int N> struct JacobiLds {
    double cs[2][N - 1][JacobiGeom<N>::PL][2];      // the rotations of a sweep, two sweeps deep
    double norm[N];
    int rank[N];
    int flag[2];
};

__device__ __forceinline__ double jacobi_swap_sum(double x, bool by32) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    const auto l = by32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                        : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = by32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                        : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __longlong_as_double((int64_t)(((uint64_t)h[0] << 32) | l[0])) +
           __longlong_as_double((int64_t)(((uint64_t)h[1] << 32) | l[1]));
}
// sum over the lanes of a pair (the lane bits above log2 PL), in every lane
template <int PL> __device__ __forceinline__ double jacobi_sum(double x) {
    if constexpr (PL == 8) x += dpp64<0x128>(x);   // row_ror:8: lane ^ 8
    x = jacobi_swap_sum(x, false);                 // lane ^ 16
    return jacobi_swap_sum(x, true);               // lane ^ 32
}

// Hands the columns on: position 0's t stays, the others move one position down
// in t, round its end into b and up in b.
template <int N> __device__ __forceinline__ void jacobi_hand_on(double& t, double& b, bool first, bool last) {
    if constexpr (N > 2) {
        const double dn = dpp64<0x101>(t), up = dpp64<0x111>(b);   // row_shl:1 (from lane + 1), row_shr:1
        t = first ? t : (last ? b : dn);
        b = first ? dn : up;
    }
}

// Rotates the pair (t, b) and hands it on.
template <int N>
__device__ __forceinline__ void jacobi_turn(double (&t)[JacobiGeom<N>::E], double (&b)[JacobiGeom<N>::E], double c,
                                            double s, bool first, bool last) {
    using G = JacobiGeom<N>;
#pragma unroll
    for (int u = 0; u < G::E; ++u) {
        double x = fma(c, t[u], -(s * b[u])), y = fma(s, t[u], c * b[u]);
        jacobi_hand_on<N>(x, y, first, last);
        t[u] = x;
        b[u] = y;
    }
}

template <int N, bool QUAD_STOP>
__device__ __forceinline__ int jacobi_left(const double* A, double* sig, double* Uo, JacobiLds<N>* J, double neg2,
                                           double quad) {
    using G = JacobiGeom<N>;
    const int lane = lane_id(), p = lane & (G::PL - 1), g = lane / G::PL;
    const bool first = p == 0, last = p == G::P - 1, in = p < G::P;
    double t[G::E], b[G::E];
#pragma unroll
    for (int u = 0; u < G::E; ++u) {
        const int e = g + G::NSUB * u;
        const bool ok = in && e < N;
        t[u] = ok ? A[p * N + e] : 0.0;
        b[u] = ok ? A[(N - 1 - p) * N + e] : 0.0;
    }
    double fro = 0.0;
#pragma unroll
    for (int u = 0; u < G::E; ++u) fro = fma(t[u], t[u], fma(b[u], b[u], fro));
    for (int off = 32; off > 0; off >>= 1) fro += __shfl_xor(fro, off, WAVE);
    // 2^-sh A has a squared norm in [1/4, 1] (sh = 0 for a zero or non-finite one)
    const int sh = (fro > 0.0 && fro < 1.7976931348623157e308) ? (ilogb(fro) + 2) >> 1 : 0;
#pragma unroll
    for (int u = 0; u < G::E; ++u) {
        t[u] = ldexp(t[u], -sh);
        b[u] = ldexp(b[u], -sh);
    }
    fro = ldexp(fro, -2 * sh);
    const double floor_abs = JACOBI_ABS * fro;
    const double floor_neg = neg2 * fro;
    const float quad_t = (float)quad;   // below it the tangent of an angle is its sine
    int sweep = 0, extra = 0;
    for (;; ++sweep) {
        float tmax = 0.f;
        double al = 0.0, be = 0.0;
#pragma unroll
        for (int u = 0; u < G::E; ++u) {
            al = fma(t[u], t[u], al);
            be = fma(b[u], b[u], be);
        }
        al = jacobi_sum<G::PL>(al);
        be = jacobi_sum<G::PL>(be);
        double* cs = &J->cs[sweep & 1][0][p][0];
        for (int rd = 0; rd < N - 1; ++rd, cs += 2 * G::PL) {
            double ga = 0.0;
#pragma unroll
            for (int u = 0; u < G::E; ++u) ga = fma(t[u], b[u], ga);
            ga = jacobi_sum<G::PL>(ga);
            // rotation by theta, |theta| <= pi/4: tan 2 theta = 2 ga / (be - al),
            // tan theta = sign(be - al) 2 ga / (|be - al| + sqrt((be - al)^2 + 4 ga^2))
            const float dl = (float)(be - al), g2 = (float)(ga + ga);
            const float hyp = __builtin_amdgcn_sqrtf(fmaf(dl, dl, g2 * g2));
            const float tn = copysignf(1.f, dl) * g2 * __builtin_amdgcn_rcpf(fabsf(dl) + hyp);
            // (lanes past the last pair hold what was handed past it: no pair)
            const bool rot = in & (ga * ga > (JACOBI_EPS * JACOBI_EPS) * (al * be)) & (fabs(ga) > floor_abs) &
                             ((al > floor_neg) | (be > floor_neg));
            const float tf = rot ? tn : 0.f;
            tmax = fmaxf(tmax, fabsf(tf));
            // one Newton step in FP64 on ga t^2 + (be - al) t - ga = 0, whose derivative at the root is +- hyp
            const double t0 = (double)tf;
            const double dt = fma(be - al, t0, ga * fma(t0, t0, -1.0)) *
                              (double)copysignf(__builtin_amdgcn_rcpf(hyp), dl);
            const double tt = rot ? t0 - dt : 0.0;
            // c = 1 / sqrt(1 + tan^2) by one third-order step from the FP32 value, s = tan c
            const double q = fma(tt, tt, 1.0);
            const double y = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.f));
            const double e = fma(-q * y, y, 1.0);
            const double c = fma(y * e, fma(0.375, e, 0.5), y), s = tt * c;
            cs[0] = c;
            cs[1] = s;
            al = fma(-tt, ga, al);
            be = fma(tt, ga, be);
            jacobi_turn<N>(t, b, c, s, first, last);
            jacobi_hand_on<N>(al, be, first, last);
        }
        bool stop = !__any(tmax > 0.f);
        if (!stop && QUAD_STOP && !__any(tmax > quad_t)) {
            stop = true;
            extra = 1;
        }
        if (!stop && sweep == JACOBI_MAX_SWEEPS - 1) {
            stop = true;
            extra = 1;
        }
        if (lane == 0) J->flag[sweep & 1] = stop ? JACOBI_LAST : JACOBI_GO;
        __syncthreads();
        if (stop) break;
    }
    // column norms, ranks (descending, ties by index), normalised outputs; the
    // columns are where they started
    double nt = 0.0, nb = 0.0;
#pragma unroll
    for (int u = 0; u < G::E; ++u) {
        nt = fma(t[u], t[u], nt);
        nb = fma(b[u], b[u], nb);
    }
    nt = sqrt(jacobi_sum<G::PL>(nt));
    nb = sqrt(jacobi_sum<G::PL>(nb));
    if (in && g == 0) {
        J->norm[p] = nt;
        J->norm[N - 1 - p] = nb;
    }
    wave_sync();
    if (lane < N) {
        // (a NaN norm ranks as infinite: the ranks are a permutation, and every entry is written)
        const double sj = J->norm[lane], kj = sj == sj ? sj : INFINITY;
        int rank = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double si = J->norm[i], ki = si == si ? si : INFINITY;
            rank += (ki > kj) || (ki == kj && i < lane);
        }
        J->rank[lane] = rank;
        sig[rank] = ldexp(sj, sh);
    }
    __syncthreads();
    if (in) {
        const int rt = J->rank[p], rb = J->rank[N - 1 - p];
        const double it = nt > 0.0 ? 1.0 / nt : 0.0, ib = nb > 0.0 ? 1.0 / nb : 0.0;
#pragma unroll
        for (int u = 0; u < G::E; ++u) {
            const int e = g + G::NSUB * u;
            if (e < N) {
                Uo[rt * N + e] = t[u] * it;
                Uo[rb * N + e] = b[u] * ib;
            }
        }
    }
    __syncthreads();
    return sweep + 1 + extra;
}

template <int N> __device__ __forceinline__ void jacobi_right(double* Vo, JacobiLds<N>* J) {
    using G = JacobiGeom<N>;
    const int lane = lane_id(), p = lane & (G::PL - 1), g = lane / G::PL;
    const bool first = p == 0, last = p == G::P - 1, in = p < G::P;
    double t[G::E], b[G::E];
#pragma unroll
    for (int u = 0; u < G::E; ++u) {
        const int e = g + G::NSUB * u;
        t[u] = (in && e == p) ? 1.0 : 0.0;
        b[u] = (in && e == N - 1 - p) ? 1.0 : 0.0;
    }
    const int pc = in ? p : 0;
    for (int sweep = 0;; ++sweep) {
        __syncthreads();
        const int flag = J->flag[sweep & 1];
#pragma unroll 2
        for (int rd = 0; rd < N - 1; ++rd)
            jacobi_turn<N>(t, b, J->cs[sweep & 1][rd][pc][0], J->cs[sweep & 1][rd][pc][1], first, last);
        if (flag == JACOBI_LAST) break;
    }
    __syncthreads();
    if (in) {
        const int rt = J->rank[p], rb = J->rank[N - 1 - p];
#pragma unroll
        for (int u = 0; u < G::E; ++u) {
            const int e = g + G::NSUB * u;
            if (e < N) {
                Vo[rt * N + e] = t[u];
                Vo[rb * N + e] = b[u];
            }
        }
    }
    __syncthreads();
}

template <int N, bool QUAD_STOP = true>
__device__ __forceinline__ int jacobi_svd(int wave, const double* A, double* sig, double* Uo, double* Vo,
                                          JacobiLds<N>* J, double neg2 = 0.0, double quad = JACOBI_QUAD) {
    if (wave == 0) return jacobi_left<N, QUAD_STOP>(A, sig, Uo, J, neg2, quad);
    if (wave == 1) {
        jacobi_right<N>(Vo, J);
        return 0;
    }
    for (int sweep = 0;; ++sweep) {
        __syncthreads();
        if (J->flag[sweep & 1] != JACOBI_GO) break;
    }
    __syncthreads();
    __syncthreads();
    return 0;
}

// ---- the update kernel's closing sums -----------------------------------------
//
// Sums of the per-workgroup partials the update kernel leaves in gpart (gU U
// side, gV V side) and what follows from them: Gram(U_f) = R_U^T R_U and
// Gram(V_f) = R_V^T R_V (R^{-1} by Cholesky, into RUinv/RVinv, or RAinv/RBinv
// for the exact bases) and, with cross, A_L^T U_f and B_L^T V_f (GAU, GBV)
// for the gather of the next rebuilding pass. The whole workgroup (NT threads)
// sums in a fixed order; its first wave factorises. Run by the update kernel's
// last workgroup when it enters from a given state, and otherwise by the first
// workgroup to finish the streaming pass that follows (ctrl->post_update).
// L: loads in flight per thread (the order of the sums, and so the result,
// does not depend on it). lds: FINISH_LDS<K, NT>() doubles of LDS scratch.
template <int K, int NT> constexpr int FINISH_LDS() { return 8 * K * K + NT; }
template <int K, int NT, int L>
__device__ __forceinline__ void finish_basis(const double* __restrict__ gpart, int gU, int gV, bool cross,
                                             bool exact, Small* sm, double* lds) {
    double* gg = lds;                 // 4 K^2: the four sums
    double* rr = gg + 4 * K * K;      // K^2 each: R_U, R_U^{-1}, R_V, R_V^{-1}
    double* ri = rr + K * K;
    double* rr2 = ri + K * K;
    double* ri2 = rr2 + K * K;
    double* part = ri2 + K * K;       // NT
    if (cross) block_sum_partials<K * K, 4, NT, L>(gpart, gU, gV, gg, part);
    else block_sum_partials<K * K, 2, NT, L>(gpart, gU, gV, gg, part);
    if (threadIdx.x < WAVE) {
        if (cross) {
            w_store<K>(gg + 2 * K * K, sm->GAU);
            w_store<K>(gg + 3 * K * K, sm->GBV);
        }
        w_chol_inv2<K>(gg, rr, ri, gg + K * K, rr2, ri2);
        w_store<K>(ri, exact ? sm->RAinv : sm->RUinv);
        w_store<K>(ri2, exact ? sm->RBinv : sm->RVinv);
    }
}

// End of a streaming-pass workgroup: workgroup 0 of the launch (of each
// instance), which starts first on its CU and is among the first to finish,
// completes the update kernel that preceded the pass when that kernel left
// its closing sums to the pass (post_update 1: Grams, 2: Grams and cross
// products). Its results are first read by the gather after the pass. The
// flag is set by the update kernel and cleared here and by every other kernel
// that overwrites the partials.
// lds: FINISH_LDS<K, NT>() doubles of the pass's LDS, free once its tile is
// done (the barrier below separates the two uses).
template <int K, int NT>
__device__ __forceinline__ void pass_finishes_update(Ctrl* ctrl, const StreamGeom& g, int64_t off, double* lds) {
    if (g.post_gpart == nullptr || blockIdx.x != 0) return;
    const int mode = ctrl->post_update;
    if (mode == 0) return;
    __syncthreads();
    // 32 loads in flight per thread, as in the update kernel: with fewer, a
    // sum over the 2 x 79 partials of m = n = 2 10^4 takes tens of dependent
    // round trips and can outlast the pass (the pass's own registers still
    // bound the kernel's)
    finish_basis<K, NT, 32>(moved(g.post_gpart, off), g.post_gU, g.post_gV, mode == 2, false,
                           moved(g.post_small, off), lds);
    if (threadIdx.x == 0) ctrl->post_update = 0;
}

}  // namespace
}  // namespace rpca
