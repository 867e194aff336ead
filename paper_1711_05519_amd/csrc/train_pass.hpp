// The pass over D of the relaxed iterations (threshold training): the forward
// step with its zeta-derivative, the recomputation of a body and the reverse
// step of the unrolled iterations.
//
// Per element, with x = D - L_k and g = logistic((|x| - zeta) / tau): z = D - x g,
// and a second quantity: dZ/dzeta = x g (1 - g) / tau (forward step), nothing
// (recomputation), or h = Zbar s'(x), Zbar = Uz Xz^T + Yz Vz^T (reverse step).
// The pass forms the products of both with thin bases over the rows and over
// the columns, in FP64.
//
// Bound by FP64 arithmetic: about 45 vector instructions for the logistic,
// and K to 3K multiply-adds per element for each of the two directions. Those
// are contractions, so they run on the FP64 matrix cores beside the vector
// ALUs (v_mfma_f64_16x16x4), in 16 x 16 blocks of D:
//   - The block is held transposed, lane l owning row l % 16 and the four
//     columns 4 (l / 16) + r: the output layout of the instruction with the
//     columns of D along its first index, numbered so that a lane's four are
//     adjacent in memory (one or two 16-byte loads). x = D - L is then one
//     accumulation onto the loaded values, Zbar another.
//   - For the sums over columns (Z V) the lane layout of the block is already
//     that of the first operand (row l % 16, k = l / 16), so no lane
//     communicates with another; for the sums over rows (Z^T U) the block
//     goes through 2 KB of the wave's own LDS once.
// A workgroup of 8 waves takes TM rows x 256 columns, 32 columns per wave, 16
// rows at a time; the column sums stay in registers over the tile, the row sums
// of the 8 waves meet in LDS (two buffers, one barrier per 16 rows). D and the
// row operands of the next 16 rows are loaded before the current ones are used.
// The reverse step's do not all fit the 256 registers that a lane of 8-wave
// workgroups has: it keeps 23 (K = 1), 49 (K = 5) or 143 (K = 9, 10) of them in
// scratch memory, in the row loop too. The other steps keep none there.
// One thread per column with a workgroup sum of every row product (two
// barriers and 6 shuffles per product and row), which this replaces, took 402
// (forward step, r = 8), 267 and 788 us (recomputation and reverse step, r = 5)
// at m = n = 2000 in FP64; now 29, 22 and 52 us.
#pragma once

#include <float.h>

#include "launch.hpp"
#include "wave.hpp"

namespace rpca {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

enum TrainMode : int { TRAIN_STEP = 0, TRAIN_RECOMPUTE = 1, TRAIN_REVERSE = 2 };

constexpr int TP_WAVES = 8;
constexpr int TP_THREADS = TP_WAVES * WAVE;
constexpr int TP_STRIPS = RX_THREADS / (16 * TP_WAVES);   // 16-column strips of a wave
constexpr int TP_PITCH = 18;                              // doubles per LDS row of a block (16-byte rows)

// A thin operand: rows or columns of D by up to 2K values, row stride ld.
template <typename TP> struct ThinRef {
    const TP* p;
    int32_t ld;
};

template <typename TP> struct TrainPass {
    const void* D;
    int64_t ldd;
    int32_t m, n, TM, n_ct, n_rt, hw;   // hw: width of the second products (reverse: K or 2K)
    double zeta, itau;                  // itau = 1 / tau
    ThinRef<TP> Lr, Lc;                 // L = Lr diag(sig) Lc^T
    const double* sig;                  // or null: 1
    ThinRef<TP> r0, c0;                 // bases of z (and of dz): sums over rows take r0, over columns c0
    ThinRef<TP> r1, c1;                 // bases of h
    ThinRef<TP> Uz, Yz, Xz, Vz;         // Zbar
    double* Rp;                         // [n_ct][m][WR], WR = K + (second products)
    double* Cp;                         // [n_rt][n][WR]
    double* scal;                       // per tile: sum (x - s)^2, sum Zbar dZ/dzeta
};

// 1 / d for a positive normal d, to about an ulp (an approximation and two Newton
// steps; a division rounds correctly, in about twice the instructions). With
// 1 / tau rounded once on the host, u = (|x| - zeta) / tau and the logistic are within
// a few roundings of the divided forms, with tanh for the logistic: m = n = 2000 in
// 64 bits, relaxed step at r = 8 2.6e-15 from its value (divided 2.6e-15), reverse
// sweep of 8 bodies at r = 5 4.1e-12 (divided 5.9e-12).
__device__ __forceinline__ double rcp64(double d) {
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    return fma(fma(-d, y, 1.0), y, y);
}

template <typename T>
__device__ __forceinline__ void tp_load_d(const T* __restrict__ p, int nv, double (&d)[4]) {
    constexpr int VW = 16 / (int)sizeof(T);
    typedef T VecT __attribute__((ext_vector_type(VW), aligned(sizeof(T))));
    if (nv == 4) {
#pragma unroll
        for (int v = 0; v < 4 / VW; ++v) {
            const VecT x = *reinterpret_cast<const VecT*>(p + v * VW);
#pragma unroll
            for (int q = 0; q < VW; ++q) d[v * VW + q] = static_cast<double>(x[q]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = q < nv ? static_cast<double>(p[q]) : 0.0;
    }
}

// p[row][c] of a thin operand of K values per row, zero from K on
template <int K, typename TP>
__device__ __forceinline__ double tp_thin(const ThinRef<TP>& t, int row, int c) {
    const double v = static_cast<double>(t.p[(size_t)row * t.ld + (c < K ? c : 0)]);
    return c < K ? v : 0.0;
}

template <typename T, typename TP, int K, int MODE>
__global__ __launch_bounds__(TP_THREADS) void k_train_pass(TrainPass<TP> a) {
    constexpr bool STEP = MODE == TRAIN_STEP, REV = MODE == TRAIN_REVERSE;
    constexpr bool SECOND = MODE != TRAIN_RECOMPUTE;
    constexpr int KS = (K + 3) / 4;                             // k steps of the rebuild
    constexpr int KZ = REV ? (2 * K + 3) / 4 : 1;               // k steps of Zbar
    constexpr int NT1 = REV ? (2 * K + 15) / 16 : (STEP ? 1 : 0);   // 16-wide blocks of the second products
    constexpr int NT1A = NT1 > 0 ? NT1 : 1;
    constexpr int WMAX = K + (STEP ? K : REV ? 2 * K : 0);
    const int w1 = STEP ? K : REV ? a.hw : 0;
    const int WR = K + w1;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lr = lane & 15, lg = lane >> 4;
    const int ct = blockIdx.x % a.n_ct, rt = blockIdx.x / a.n_ct;
    const int c0 = ct * RX_THREADS + 16 * TP_STRIPS * wave;
    const int i_lo = rt * a.TM, i_hi = min(a.m, i_lo + a.TM);
    const T* __restrict__ D = static_cast<const T*>(a.D);
    const double zeta = a.zeta, itau = a.itau;

    __shared__ double blk[TP_WAVES][16 * TP_PITCH];
    __shared__ double rows[2][TP_WAVES][16 * WMAX];
    __shared__ double red[TP_WAVES];

    // Column operands of the wave's strips. Rows and columns past the matrix
    // repeat the last one: their z and h are set to zero below.
    double ca[TP_STRIPS][KS], cz[TP_STRIPS][KZ], cb[TP_STRIPS][4], ch[TP_STRIPS][NT1A][4];
    int jb[TP_STRIPS], nv[TP_STRIPS];
#pragma unroll
    for (int s = 0; s < TP_STRIPS; ++s) {
        const int base = c0 + 16 * s;
        jb[s] = base + 4 * lg;
        nv[s] = min(max(a.n - jb[s], 0), 4);
        const int cA = min(base + 4 * (lr & 3) + (lr >> 2), a.n - 1);   // column of first-operand line lr
#pragma unroll
        for (int q = 0; q < KS; ++q) ca[s][q] = tp_thin<K>(a.Lc, cA, lg + 4 * q);
        if constexpr (REV) {
#pragma unroll
            for (int q = 0; q < KZ; ++q) {
                const int k = lg + 4 * q;
                cz[s][q] = k < K ? tp_thin<K>(a.Xz, cA, k) : tp_thin<K>(a.Vz, cA, k - K);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = min(jb[s] + r, a.n - 1);
            cb[s][r] = tp_thin<K>(a.c0, col, lr);
            if constexpr (REV) {
#pragma unroll
                for (int t = 0; t < NT1; ++t) {
                    const int c = 16 * t + lr;
                    const double v = static_cast<double>(a.c1.p[(size_t)col * a.c1.ld + (c < w1 ? c : 0)]);
                    ch[s][t][r] = c < w1 ? v : 0.0;
                }
            }
        }
    }
    double sg[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        const int k = lg + 4 * q;
        sg[q] = k < K ? (a.sig ? -a.sig[k] : -1.0) : 0.0;
    }

    f64x4 y2[TP_STRIPS], y2h[TP_STRIPS][NT1A];
#pragma unroll
    for (int s = 0; s < TP_STRIPS; ++s) {
        y2[s] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < NT1A; ++t) y2h[s][t] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    double res = 0.0, zsum = 0.0;

    // operands of 16 rows: D, and the thin rows
    struct Rows {
        double d[TP_STRIPS][4], l[KS], b0[4], b1[NT1A][4], z[KZ];
    };
    auto load = [&](int ib, Rows& R) {
        const int row = min(ib + lr, a.m - 1);
#pragma unroll
        for (int s = 0; s < TP_STRIPS; ++s)
            tp_load_d<T>(D + (size_t)row * a.ldd + jb[s], ib + lr < a.m ? nv[s] : 0, R.d[s]);
#pragma unroll
        for (int q = 0; q < KS; ++q) R.l[q] = tp_thin<K>(a.Lr, row, lg + 4 * q);
        if constexpr (REV) {
#pragma unroll
            for (int q = 0; q < KZ; ++q) {
                const int k = lg + 4 * q;
                R.z[q] = k < K ? tp_thin<K>(a.Uz, row, k) : tp_thin<K>(a.Yz, row, k - K);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rq = min(ib + lg + 4 * q, a.m - 1);
            R.b0[q] = tp_thin<K>(a.r0, rq, lr);
            if constexpr (REV) {
#pragma unroll
                for (int t = 0; t < NT1; ++t) {
                    const int c = 16 * t + lr;
                    const double v = static_cast<double>(a.r1.p[(size_t)rq * a.r1.ld + (c < w1 ? c : 0)]);
                    R.b1[t][q] = c < w1 ? v : 0.0;
                }
            }
        }
    };

    Rows cur, nxt;
    if (i_lo < i_hi) load(i_lo, nxt);
    int buf = 0;
    for (int ib = i_lo; ib < i_hi; ib += 16, buf ^= 1) {
        cur = nxt;
        if (ib + 16 < i_hi) load(ib + 16, nxt);
        const bool rok = ib + lr < a.m;
        f64x4 y1 = {0.0, 0.0, 0.0, 0.0}, y1h[NT1A];
#pragma unroll
        for (int t = 0; t < NT1A; ++t) y1h[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < TP_STRIPS; ++s) {
            f64x4 x = {cur.d[s][0], cur.d[s][1], cur.d[s][2], cur.d[s][3]};
#pragma unroll
            for (int q = 0; q < KS; ++q)
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[s][q], cur.l[q] * sg[q], x, 0, 0, 0);
            f64x4 zb = {0.0, 0.0, 0.0, 0.0};
            if constexpr (REV) {
#pragma unroll
                for (int q = 0; q < KZ; ++q)
                    zb = __builtin_amdgcn_mfma_f64_16x16x4f64(cz[s][q], cur.z[q], zb, 0, 0, 0);
            }
            double z[4], h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double ax = fabs(x[r]);
                const double u = (ax - zeta) * itau;
                // logistic(u) and 1 - logistic(u), each to FP64 accuracy: exp(-|u|) cannot overflow
                const double e = exp(-fabs(u));
                const double p = rcp64(1.0 + e), ep = e * p;
                const double g = u >= 0.0 ? p : ep, og = u >= 0.0 ? ep : p;
                const bool ok = rok && r < nv[s];
                const double ex = x[r] * og;   // x - s(x)
                if (ok) res = fma(ex, ex, res);
                z[r] = ok ? cur.d[s][r] - x[r] * g : 0.0;
                if constexpr (SECOND) {
                    const double gg = p * ep * itau;   // g (1 - g) / tau
                    if constexpr (STEP) {
                        h[r] = ok ? x[r] * gg : 0.0;
                    } else {
                        if (ok) zsum = fma(zb[r], x[r] * gg, zsum);
                        h[r] = ok ? zb[r] * fma(ax, gg, g) : 0.0;
                    }
                }
            }
            // sums over the columns: the block is the first operand as it lies
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y1 = __builtin_amdgcn_mfma_f64_16x16x4f64(z[r], cb[s][r], y1, 0, 0, 0);
                if constexpr (STEP) y1h[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(h[r], cb[s][r], y1h[0], 0, 0, 0);
                if constexpr (REV) {
#pragma unroll
                    for (int t = 0; t < NT1; ++t)
                        y1h[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(h[r], ch[s][t][r], y1h[t], 0, 0, 0);
                }
            }
            // sums over the rows: the block transposed through the wave's LDS
            double* b = blk[wave];
#pragma unroll
            for (int second = 0; second < (SECOND ? 2 : 1); ++second) {
                const double(&v)[4] = second ? h : z;
#pragma unroll
                for (int r = 0; r < 4; ++r) b[lr * TP_PITCH + 4 * lg + r] = v[r];
                wave_sync();
                double w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) w[q] = b[(lg + 4 * q) * TP_PITCH + lr];
                wave_sync();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (second == 0) {
                        y2[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[q], cur.b0[q], y2[s], 0, 0, 0);
                    } else if constexpr (STEP) {
                        y2h[s][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[q], cur.b0[q], y2h[s][0], 0, 0, 0);
                    } else if constexpr (REV) {
#pragma unroll
                        for (int t = 0; t < NT1; ++t)
                            y2h[s][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[q], cur.b1[t][q], y2h[s][t], 0, 0, 0);
                    }
                }
            }
        }
        // row sums of the 8 waves, in wave order
        double* mine = rows[buf][wave];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = lg + 4 * r;
            if (lr < K) mine[row * WMAX + lr] = y1[r];
#pragma unroll
            for (int t = 0; t < NT1; ++t)
                if (16 * t + lr < w1) mine[row * WMAX + K + 16 * t + lr] = y1h[t][r];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 16 * WR; e += TP_THREADS) {
            const int row = e / WR, c = e - row * WR;
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < TP_WAVES; ++w) v += rows[buf][w][row * WMAX + c];
            if (ib + row < i_hi) a.Rp[((size_t)ct * a.m + ib + row) * WR + c] = v;
        }
    }
#pragma unroll
    for (int s = 0; s < TP_STRIPS; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = c0 + 16 * s + lg + 4 * r;
            if (col >= a.n) continue;
            double* out = a.Cp + ((size_t)rt * a.n + col) * WR;
            if (lr < K) out[lr] = y2[s][r];
#pragma unroll
            for (int t = 0; t < NT1; ++t)
                if (16 * t + lr < w1) out[K + 16 * t + lr] = y2h[s][t][r];
        }
    const double r1 = block_sum(res, red);
    const double r2 = REV ? block_sum(zsum, red) : 0.0;
    if (threadIdx.x == 0) {
        a.scal[2 * blockIdx.x] = r1;
        a.scal[2 * blockIdx.x + 1] = r2;
    }
}

}  // namespace
}  // namespace rpca
