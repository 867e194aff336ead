// Thin-panel steps between the training passes: FP64 panels of m (U side) or n
// (V side) rows and up to 46 columns.
//
// One launch does, for both sides at once,
//   sum      tile partials of a pass into a panel, in tile order;
//   combine  out = [panels] S with a small S, optionally followed by a row-wise
//            Trim (Algorithm 2) or its reverse;
//   gram     G = [panels]^T [panels] over the rows;
//   tail     small dense algebra on the Grams, by the last workgroup.
// Each part is optional; a later part reads what an earlier one wrote for the
// same rows.
//
// Bound by latency (a 2000 x 5 panel is 80 KB): a step is a launch, a few
// dependent loads, the election of the last workgroup and the tail, so what
// counts is how many launches a body takes and that each part's loads are
// issued together. Both contractions run on v_mfma_f64_16x16x4 by 16-row
// blocks, one block per wave: the output layout of a combination (row l / 16 +
// 4 r, column l % 16) is the operand layout of a Gram step, and no operand goes
// through LDS. As separate kernels (sum, Gram by one thread per entry, one-wave
// tails, one thread per combined entry) a body of the reverse sweep took 30
// launches and a relaxed step 6; now 12 and 3. At m = n = 2000 in FP64 the
// panel work of a reverse body at r = 5 went from 390 to 165 us, that of a
// relaxed step at r = 8 from 255 to 120 us.
#pragma once

#include <initializer_list>

#include "launch.hpp"
#include "wave.hpp"

namespace rpca {
namespace {

typedef double panel4 __attribute__((ext_vector_type(4)));

constexpr int TR_NPAN = 4;                // panels side by side
constexpr int TR_T = 3;                   // 16-column blocks of a Gram's sides: 48 columns
constexpr int TR_TILES = 6;               // blocks of a Gram
constexpr int TR_CT = 2;                  // 16-column blocks of a combination: 32 columns

// A panel: w columns of rows with stride ld, FP64 or (f32) FP32 values.
struct PanelRef {
    const void* p;
    int32_t ld, w, f32;
};

struct SumJob {               // out[row][c] = sum over tiles of part[tile][row][c], c < W
    const double* part;       // null: no sum
    double* out;
    int32_t tiles, W;
    PanelRef add;             // add.w > 0: out2 = (the first add.w columns of out) + add
    double* out2;
};

enum RowPost : int { POST_NONE = 0, POST_TRIM = 1, POST_TRIM_REVERSE = 2 };

struct CombJob {              // out = [in] S; nin = 0 with POST_TRIM: out = Trim(X)
    PanelRef in[TR_NPAN];
    int32_t nin, win, q, ldo;
    const double* S;          // win x q, row-major
    double* out;              // null: no combination
    int32_t post, K;          // Trim: rows of X scaled by min(1, c / ||row||)
    const double* X;          // m x K
    double c;                 // trim level; <= 0: no trim
};

struct GramJob {              // out = [L]^T [R], wL x wR row-major
    PanelRef L[TR_NPAN], R[TR_NPAN];
    int32_t nL, nR, wL, wR;
    double* out;              // null: no Gram
};

struct SideJob {
    int32_t rows, nblk, per;  // per: rows per workgroup (a multiple of TR_ROWS)
    SumJob sum;
    CombJob comb;
    GramJob gram;
};

template <typename TailArgs> struct StepArgs {
    SideJob side[2];
    const double* scal;       // per-tile pairs of a pass; scal_out = sum of the second values (null: none)
    double* scal_out;
    int32_t tiles;
    double* gpart;
    uint32_t* cnt;
    TailArgs tail;
};

// The panel and column holding column c of the concatenation (null past its end).
__device__ __forceinline__ void panel_at(const PanelRef* P, int np, int c, const char*& p, int& ld, bool& f32) {
    p = nullptr;
    ld = 0;
    f32 = false;
    for (int q = 0; q < np; ++q) {
        if (c >= 0 && c < P[q].w) {
            f32 = P[q].f32 != 0;
            p = static_cast<const char*>(P[q].p) + (size_t)c * (f32 ? 4 : 8);
            ld = P[q].ld;
        }
        c -= P[q].w;
    }
}
__device__ __forceinline__ double panel_load(const char* p, int ld, bool f32, int row) {
    const size_t o = (size_t)row * ld;
    return f32 ? static_cast<double>(reinterpret_cast<const float*>(p)[o]) : reinterpret_cast<const double*>(p)[o];
}

// One 16-row block of a combination, by one wave. The rows ib .. ib + 15 are
// clamped to the panel; stores are not.
__device__ __forceinline__ void comb_block(const CombJob& J, int rows, int ib) {
    const int lane = lane_id(), lr = lane & 15, lg = lane >> 4;
    panel4 v[TR_CT];
#pragma unroll
    for (int u = 0; u < TR_CT; ++u) v[u] = panel4{0.0, 0.0, 0.0, 0.0};
    const int arow = min(ib + lr, rows - 1);
    constexpr int U = 4;   // k steps whose loads are in flight together
    for (int q0 = 0; 4 * q0 < J.win; q0 += U) {
        double a[U], b[TR_CT][U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int k = 4 * (q0 + q) + lg;
            const char* p;
            int ld;
            bool f32;
            panel_at(J.in, J.nin, k, p, ld, f32);
            a[q] = p ? panel_load(p, ld, f32, arow) : 0.0;
#pragma unroll
            for (int u = 0; u < TR_CT; ++u) {
                const int c = 16 * u + lr;
                b[u][q] = (k < J.win && c < J.q) ? J.S[k * J.q + c] : 0.0;
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
            for (int u = 0; u < TR_CT; ++u)
                if (16 * u < J.q) v[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[u][q], v[u], 0, 0, 0);
    }
    if (J.post != POST_NONE) {
        const int c = lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = min(ib + lg + 4 * r, rows - 1);
            const double x = c < J.K ? J.X[(size_t)row * J.K + c] : 0.0;
            const double rho = sqrt(row16_sum(x * x));
            const bool big = J.c > 0.0 && rho > J.c;
            const double w = big ? J.c / rho : 1.0;
            if (J.post == POST_TRIM) {
                v[0][r] = w * x;
            } else {
                // Xbar = w Abar - [rho > c] (c / rho^3) (Abar . x) x
                const double ab = c < J.K ? v[0][r] : 0.0;
                const double dot = row16_sum(ab * x);
                const double f = big ? J.c / (rho * rho * rho) * dot : 0.0;
                v[0][r] = fma(w, ab, -f * x);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < TR_CT; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = ib + lg + 4 * r, c = 16 * u + lr;
            if (row < rows && c < J.q) J.out[(size_t)row * J.ldo + c] = v[u][r];
        }
}

// Tail: a struct with Args and static run(const Args&), called by all threads of
// the last workgroup once the Grams are in memory; Args::none() skips it.
template <typename Tail>
__global__ __launch_bounds__(TR_THREADS) void k_train_rows(StepArgs<typename Tail::Args> a) {
    const int side = (int)blockIdx.x < a.side[0].nblk ? 0 : 1;
    const SideJob& J = a.side[side];
    const int b = side ? (int)blockIdx.x - a.side[0].nblk : (int)blockIdx.x;
    const int r_lo = b * J.per, r_hi = min(J.rows, r_lo + J.per);
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lr = lane & 15, lg = lane >> 4;
    __shared__ double tiles[TR_WAVES][TR_TILES * 256];
    __shared__ int flag;

    if (J.sum.part) {
        // the workgroup's rows are one contiguous block of every tile's partial
        const int W = J.sum.W;
        const size_t stride = (size_t)J.rows * W;
        const int cnt = (r_hi - r_lo) * W;
        const double* part = J.sum.part + (size_t)r_lo * W;
        for (int e = threadIdx.x; e < cnt; e += TR_THREADS) {
            double v = 0.0;
            int t = 0;
            for (; t + 8 <= J.sum.tiles; t += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = part[(size_t)(t + u) * stride + e];
#pragma unroll
                for (int u = 0; u < 8; ++u) v += x[u];
            }
            for (; t < J.sum.tiles; ++t) v += part[(size_t)t * stride + e];
            J.sum.out[(size_t)r_lo * W + e] = v;
            if (J.sum.add.w > 0) {
                const int row = r_lo + e / W, c = e % W;
                if (c < J.sum.add.w)
                    J.sum.out2[(size_t)row * J.sum.add.w + c] =
                        v + static_cast<const double*>(J.sum.add.p)[(size_t)row * J.sum.add.ld + c];
            }
        }
        __syncthreads();
    }
    if (a.scal && blockIdx.x == 0) {
        double v = 0.0;
        for (int t = threadIdx.x; t < a.tiles; t += TR_THREADS) v += a.scal[2 * t + 1];
        v = block_sum(v, &tiles[0][0]);
        if (threadIdx.x == 0) *a.scal_out = v;
        __syncthreads();
    }
    if (J.comb.out) {
        for (int ib = r_lo + 16 * wave; ib < r_hi; ib += TR_ROWS) comb_block(J.comb, J.rows, ib);
        __syncthreads();
    }
    if (!a.side[0].gram.out && !a.side[1].gram.out) return;

    const GramJob& G = J.gram;
    const int nTL = (G.wL + 15) / 16, nTR = (G.wR + 15) / 16;
    panel4 acc[TR_T][TR_T];
#pragma unroll
    for (int i = 0; i < TR_T; ++i)
#pragma unroll
        for (int j = 0; j < TR_T; ++j) acc[i][j] = panel4{0.0, 0.0, 0.0, 0.0};
    if (G.out) {
        const char *pl[TR_T], *pq[TR_T];
        int ll[TR_T], lq[TR_T];
        bool fl[TR_T], fq[TR_T];
#pragma unroll
        for (int t = 0; t < TR_T; ++t) {
            panel_at(G.L, G.nL, 16 * t + lr, pl[t], ll[t], fl[t]);
            panel_at(G.R, G.nR, 16 * t + lr, pq[t], lq[t], fq[t]);
        }
        for (int ib = r_lo + 16 * wave; ib < r_hi; ib += TR_ROWS) {
            double x[TR_T][4], y[TR_T][4];
#pragma unroll
            for (int t = 0; t < TR_T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = ib + lg + 4 * r;
                    x[t][r] = (row < r_hi && pl[t]) ? panel_load(pl[t], ll[t], fl[t], row) : 0.0;
                    y[t][r] = (row < r_hi && pq[t]) ? panel_load(pq[t], lq[t], fq[t], row) : 0.0;
                }
#pragma unroll
            for (int i = 0; i < TR_T; ++i)
#pragma unroll
                for (int j = 0; j < TR_T; ++j) {
                    if (i >= nTL || j >= nTR) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][r], y[j][r], acc[i][j], 0, 0, 0);
                }
        }
#pragma unroll
        for (int i = 0; i < TR_T; ++i)
#pragma unroll
            for (int j = 0; j < TR_T; ++j) {
                if (i >= nTL || j >= nTR) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) tiles[wave][(i * nTR + j) * 256 + (lg + 4 * r) * 16 + lr] = acc[i][j][r];
            }
        __syncthreads();
        double* gp = a.gpart + (size_t)blockIdx.x * TR_GE;
        for (int e = threadIdx.x; e < G.wL * G.wR; e += TR_THREADS) {
            const int i = e / G.wR, j = e - i * G.wR;
            const int at = ((i >> 4) * nTR + (j >> 4)) * 256 + (i & 15) * 16 + (j & 15);
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < TR_WAVES; ++w) v += tiles[w][at];
            store_agent(gp + e, v);
        }
    }
    if (!last_block_arrives(a.cnt, &flag)) return;
    for (int s = 0; s < 2; ++s) {
        const SideJob& Q = a.side[s];
        if (!Q.gram.out) continue;
        const double* gp = a.gpart + (size_t)(s ? a.side[0].nblk : 0) * TR_GE;
        for (int e = threadIdx.x; e < Q.gram.wL * Q.gram.wR; e += TR_THREADS) {
            double v = 0.0;
            for (int t = 0; t < Q.nblk; t += 16) {
                double x[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) x[u] = t + u < Q.nblk ? gp[(size_t)(t + u) * TR_GE + e] : 0.0;
#pragma unroll
                for (int u = 0; u < 16; ++u) v += x[u];
            }
            Q.gram.out[e] = v;
        }
    }
    if (threadIdx.x == 0) *a.cnt = 0;
    __syncthreads();
    Tail::run(a.tail);
}

// ---- host side -------------------------------------------------------------------

inline PanelRef panel_ref(const void* p, int ld, int w, bool f32 = false) {
    PanelRef r;
    r.p = p;
    r.ld = ld;
    r.w = w;
    r.f32 = f32 ? 1 : 0;
    return r;
}

inline void step_rows(SideJob* J, int rows) {
    J->rows = rows;
    J->per = train_rows_per_block(rows);
    J->nblk = (rows + J->per - 1) / J->per;
}

inline void step_comb(SideJob* J, std::initializer_list<PanelRef> in, const double* S, int q, double* out, int ldo) {
    for (const PanelRef& r : in) {
        J->comb.in[J->comb.nin++] = r;
        J->comb.win += r.w;
    }
    J->comb.S = S;
    J->comb.q = q;
    J->comb.out = out;
    J->comb.ldo = ldo;
}

inline void step_gram(SideJob* J, std::initializer_list<PanelRef> L, std::initializer_list<PanelRef> R, double* out) {
    for (const PanelRef& r : L) {
        J->gram.L[J->gram.nL++] = r;
        J->gram.wL += r.w;
    }
    for (const PanelRef& r : R) {
        J->gram.R[J->gram.nR++] = r;
        J->gram.wR += r.w;
    }
    J->gram.out = out;
}

inline void step_sum(SideJob* J, const double* part, int tiles, int W, double* out) {
    J->sum.part = part;
    J->sum.tiles = tiles;
    J->sum.W = W;
    J->sum.out = out;
}

// What the kernel's fixed sizes assume of a step.
template <typename A> bool step_fits(const StepArgs<A>& a) {
    for (const SideJob& J : a.side) {
        const int tl = (J.gram.wL + 15) / 16, tr = (J.gram.wR + 15) / 16;
        if (tl > TR_T || tr > TR_T || tl * tr > TR_TILES || J.gram.wL * J.gram.wR > TR_GE) return false;
        if (J.comb.q > 16 * TR_CT || J.comb.win * J.comb.q > TR_GE) return false;
        if (J.comb.post != POST_NONE && (J.comb.K > 16 || J.comb.q != J.comb.K)) return false;
    }
    return true;
}

template <typename Tail> hipError_t launch_step(const StepArgs<typename Tail::Args>& a, hipStream_t s) {
    if (!step_fits(a)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_train_rows<Tail>), dim3((unsigned)(a.side[0].nblk + a.side[1].nblk)), dim3(TR_THREADS), 0, s, a);
    return hipGetLastError();
}

}  // namespace
}  // namespace rpca
