// One AccAltProj iteration with a relaxed threshold and the derivative of a
// loss of the next iterate with respect to the threshold (training of a
// learned threshold schedule; not part of the paper).
//
// From L_k = U diag(sigma) V^T, with x = D - L_k and the relaxation
//   s(x) = x * logistic((|x| - zeta) / tau)       (T_zeta as tau -> 0)
// the iteration forms Z = D - s(x), P_T(Z) on the tangent space of Trim(L_k)
// (Section 2.1) and L_{k+1} = H_r(P_T(Z)). Its derivative in zeta is
//   dZ = dZ/dzeta = x * g (1 - g) / tau,  g = logistic((|x| - zeta) / tau),
// P_T is linear, and H_r moves by its first-order perturbation. Both P_T(Z)
// and P_T(dZ) lie in span[U*, W1, dW1] x span[V*, W2, dW2] (W, dW the
// complements of Z V* and dZ V*), a 3r x 3r reduced space with orthonormal
// bases B_U, B_V, so
//   L_{k+1} = B_U H_r(M) B_V^T,   dL_{k+1} = B_U U_M F V_M^T B_V^T
// with M, dM the 3r x 3r reductions, M = U_M S V_M^T, E = U_M^T dM V_M and
//   F_ij = E_ij (i, j < r);  F_ij = (s_i^2 E_ij + s_i s_j E_ji) / (s_i^2 - s_j^2),
//   F_ji = (s_i^2 E_ji + s_i s_j E_ij) / (s_i^2 - s_j^2)  (i < r <= j);  0 else.
// The loss is ||L_{k+1} - P Q^T||_F^2 / ||P Q^T||_F^2 for given factors P, Q
// (the ground truth of a synthetic instance); it and its derivative need only
// projections of P and Q onto B_U and B_V.
//
// Kernels: one pass over D giving [Y1 dY1] = [Z dZ] V_f and [Y2 dY2] = [Z dZ]^T U_f
// as per-tile partials (plus the relaxed residual; train_pass.hpp), then three
// panel steps (train_panel.hpp): the sums over the tiles with the products
// [U_f | P]^T [Y1 dY1 | P] (for C, dC and U*^T P); the explicit complements
// [W1 dW1] = [Y1 dY1] R_V^{-1} - U* [C dC] (and the V side), formed row by row
// in FP64 as the FP64 loop path does (Gram differences would cancel), with
// their exact Grams and the small FP64 algebra; and the new factors.

#include <math.h>
#include <string.h>

#include <initializer_list>

#include "launch.hpp"
#include "train_panel.hpp"
#include "train_pass.hpp"
#include "wave.hpp"

namespace rpca {
namespace {

template <typename T> inline const T* cptr(const void* p) { return static_cast<const T*>(p); }

struct RelaxTailArgs {
    int32_t stage, rt;            // 1: after the first Grams, 2: after the second
    const double* G1[2];          // [F | P]^T [Y dY | P], (K + rt) x (2K + rt), U side and V side
    const double* G2[2];          // [W dW]^T [W dW | P], 2K x (2K + rt)
    const double* Rinv[2];        // R_U^{-1}, R_V^{-1} (row stride KMAX)
    double* S[2];                 // stage 1: coefficients of the complements (3K x 2K); stage 2: of the factors (3K x K)
    double* C;                    // C, then dC (K x K each)
    const double* scal;           // per-tile residuals of the pass (pairs)
    int32_t tiles;
    double normD2;
    double* sigma_out;
    RelaxResult* result;
};

// The small FP64 algebra, by the last workgroup of a panel step.
template <int K> struct RelaxTail {
    using Args = RelaxTailArgs;
    static constexpr int K2 = 2 * K, K3 = 3 * K;

    // C = Ra^T (F^T Y) Rb and dC = Ra^T (F^T dY) Rb; the complements' coefficients
    // for [Y dY | F]: [W dW] = [Y dY] diag(Rb, Rb) - F Ra [C dC]
    static __device__ __forceinline__ void stage1(const Args& a) {
        __shared__ double ra[K * K], rb[K * K], g[2 * K * K], t[2 * K * K], c[2 * K * K];
        const int tid = threadIdx.x;
        const int wR = K2 + a.rt;
        for (int side = 0; side < 2; ++side) {
            for (int e = tid; e < K * K; e += TR_THREADS) {
                ra[e] = a.Rinv[side][(e / K) * KMAX + e % K];
                rb[e] = a.Rinv[1 - side][(e / K) * KMAX + e % K];
            }
            for (int e = tid; e < 2 * K * K; e += TR_THREADS) g[e] = a.G1[side][(e / K2) * wR + e % K2];   // K x 2K
            __syncthreads();
            for (int e = tid; e < 2 * K * K; e += TR_THREADS) {   // t = (F^T [Y dY]) diag(Rb, Rb)
                const int i = e / K2, j = e % K2, w = j / K;
                double v = 0.0;
                for (int l = 0; l < K; ++l) v = fma(g[i * K2 + w * K + l], rb[l * K + j - w * K], v);
                t[e] = v;
            }
            __syncthreads();
            for (int e = tid; e < 2 * K * K; e += TR_THREADS) {   // c = Ra^T t
                const int i = e / K2, j = e % K2;
                double v = 0.0;
                for (int l = 0; l < K; ++l) v = fma(ra[l * K + i], t[l * K2 + j], v);
                c[e] = v;
                if (side == 0) a.C[(j / K) * K * K + i * K + j % K] = v;
            }
            __syncthreads();
            for (int e = tid; e < K3 * K2; e += TR_THREADS) {
                const int r = e / K2, j = e % K2;
                double v = 0.0;
                if (r < K2) {
                    if (r / K == j / K) v = rb[(r % K) * K + j % K];
                } else {
                    for (int l = 0; l < K; ++l) v = fma(ra[(r - K2) * K + l], c[l * K2 + j], v);
                    v = -v;
                }
                a.S[side][e] = v;
            }
            __syncthreads();
        }
    }

    // The reduced M and dM, the loss and its derivative, and the coefficients
    // of the new factors.
    //
    // The Cholesky factors of the Grams of [W dW] are upper triangular, so the
    // columns of M beyond 2K and its rows beyond 2K are zero: its SVD is that of the
    // leading 2K x 2K block, completed by V_j = e_j and sigma_j = 0. Singular
    // values at the rounding level are zero too, and their left vectors
    // (undefined in the one-sided method) are dropped; the left null space
    // then enters through a projector term (in the formula the block
    // j >= rank, i < K, with F_ji = E_ji). The loss needs only inner products:
    // <H, dH> = sum_i s_i F_ii, <H, P Q^T> and <dH, P Q^T> through the projections
    // a = U_M^T B_U^T P and b = V_M^T B_V^T Q.
    static __device__ __forceinline__ void stage2(const Args& a) {
        constexpr int N = K2;
        __shared__ double RG[2][K2 * K2], Ri[2][K2 * K2], GG[2][K2 * K2];
        __shared__ double ra[2][K * K], cb[2][K2];
        __shared__ double Um[N * N], Vm[N * N], sg[N];
        __shared__ JacobiLds<N> jac;
        __shared__ double dM[K3 * K3], A1[K3 * K], EL[N * K], A2[K * K3], ET[K * K3];
        __shared__ double pr[2][K3 * RX_TRUE_MAX], ab[2][K3 * RX_TRUE_MAX];
        __shared__ double red[TR_WAVES];
        __shared__ int sweeps_s;
        const int tid = threadIdx.x, rT = a.rt, wR = K2 + rT;
        for (int e = tid; e < 2 * K2 * K2; e += TR_THREADS) {
            const int side = e / (K2 * K2), i = e % (K2 * K2);
            GG[side][i] = a.G2[side][(i / K2) * wR + i % K2];
        }
        for (int e = tid; e < 2 * K * K; e += TR_THREADS) {
            const int side = e / (K * K), i = e % (K * K);
            ra[side][i] = a.Rinv[side][(i / K) * KMAX + i % K];
        }
        __syncthreads();
        if (tid < 2 * WAVE) chol_group<K2>(GG[tid / WAVE], RG[tid / WAVE], Ri[tid / WAVE], cb[tid / WAVE], lane_id());
        __syncthreads();
        // M (leading block, column-major, into GG[0], free now) and dM (row-major)
        double* M = GG[0];
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int col = e / N, row = e % N;
            double v = 0.0;
            if (row < K && col < K) v = a.C[row * K + col];
            else if (row < K) v = RG[1][(col - K) * K2 + row];
            else if (col < K) v = RG[0][(row - K) * K2 + col];
            M[e] = v;
        }
        for (int e = tid; e < K3 * K3; e += TR_THREADS) {
            const int row = e / K3, col = e % K3;
            double v = 0.0;
            if (row < K && col < K) v = a.C[K * K + row * K + col];
            else if (row < K) v = RG[1][(col - K) * K2 + K + row];
            else if (col < K) v = RG[0][(row - K) * K2 + K + col];
            dM[e] = v;
        }
        // projections B_U^T P = [R_U^{-T} (U_f^T P) ; R_G^{-T} ([W1 dW1]^T P)], likewise B_V^T Q
        for (int e = tid; e < 2 * K3 * rT; e += TR_THREADS) {
            const int side = e / (K3 * rT), x = e % (K3 * rT), i = x / rT, q = x % rT;
            double v = 0.0;
            if (i < K) {
                for (int l = 0; l < K; ++l) v = fma(ra[side][l * K + i], a.G1[side][l * wR + K2 + q], v);
            } else {
                for (int l = 0; l < K2; ++l) v = fma(Ri[side][l * K2 + i - K], a.G2[side][l * wR + K2 + q], v);
            }
            pr[side][i * rT + q] = v;
        }
        __syncthreads();
        const int sweeps = jacobi_svd<N, false>(tid / WAVE, M, sg, Um, Vm, &jac);   // Um, Vm column-major
        if (tid < WAVE) {
            const double cut = 1e-12 * sg[0];
            for (int e = tid; e < N * N; e += WAVE)
                if (sg[e / N] <= cut) Um[e] = 0.0;
            wave_sync();
            if (tid < N && sg[tid] <= cut) sg[tid] = 0.0;
            if (tid == 0) sweeps_s = sweeps;
        }
        __syncthreads();
        // A1 = dM V_K, A2 = U_K^T dM, a = U^T pr_U, b = V^T pr_V
        for (int e = tid; e < K3 * K; e += TR_THREADS) {
            const int r = e / K, t = e % K;
            double v = 0.0;
            for (int c = 0; c < N; ++c) v = fma(dM[r * K3 + c], Vm[t * N + c], v);
            A1[e] = v;
        }
        for (int e = tid; e < K * K3; e += TR_THREADS) {
            const int i = e / K3, c = e % K3;
            double v = 0.0;
            for (int r = 0; r < N; ++r) v = fma(Um[i * N + r], dM[r * K3 + c], v);
            A2[e] = v;
        }
        for (int e = tid; e < 2 * K3 * rT; e += TR_THREADS) {
            const int side = e / (K3 * rT), x = e % (K3 * rT), j = x / rT, q = x % rT;
            const double* X = side ? Vm : Um;
            double v = 0.0;
            if (j < N) {
                for (int r = 0; r < N; ++r) v = fma(X[j * N + r], pr[side][r * rT + q], v);
            } else if (side) {
                v = pr[1][j * rT + q];
            }
            ab[side][j * rT + q] = v;
        }
        __syncthreads();
        // E = U_M^T dM V_M where i < K or j < K: EL (columns j < K), ET (rows i < K)
        for (int e = tid; e < N * K; e += TR_THREADS) {
            const int i = e / K, t = e % K;
            double v = 0.0;
            for (int r = 0; r < N; ++r) v = fma(Um[i * N + r], A1[r * K + t], v);
            EL[e] = v;
        }
        for (int e = tid; e < K * K3; e += TR_THREADS) {
            const int i = e / K3, j = e % K3;
            double v = 0.0;
            if (j < N) {
                for (int c = 0; c < N; ++c) v = fma(A2[i * K3 + c], Vm[j * N + c], v);
            } else {
                v = A2[i * K3 + j];
            }
            ET[e] = v;
        }
        __syncthreads();
        double acc = 0.0, h2 = 0.0, hpq = 0.0, hdh = 0.0, hdpq = 0.0, rs = 0.0;
        auto dot = [&](const double* x, const double* y) {
            double v = 0.0;
            for (int q = 0; q < rT; ++q) v = fma(x[q], y[q], v);
            return v;
        };
        for (int b = tid; b < a.tiles; b += TR_THREADS) rs += a.scal[2 * b];   // the relaxed residual
        for (int e = tid; e < rT * rT; e += TR_THREADS) {   // ||P Q^T||^2 = tr((P^T P)(Q^T Q))
            const int at = (K + e / rT) * wR + K2 + e % rT;
            acc = fma(a.G1[0][at], a.G1[1][at], acc);
        }
        for (int e = tid; e < K * K3; e += TR_THREADS) {
            const int i = e / K3, j = e % K3;
            const double si = sg[i];
            if (j < K) {
                const double f = ET[e];
                hdpq = fma(f, dot(ab[0] + i * rT, ab[1] + j * rT), hdpq);
                if (i == j) {
                    hdh = fma(si, f, hdh);
                    h2 = fma(si, si, h2);
                    hpq = fma(si, dot(ab[0] + i * rT, ab[1] + i * rT), hpq);
                }
            } else {
                const double sj = j < N ? sg[j] : 0.0, eij = ET[e], eji = j < N ? EL[j * K + i] : 0.0;
                const double den = si * si - sj * sj;
                const double fij = (si * si * eij + si * sj * eji) / den, fji = (si * si * eji + si * sj * eij) / den;
                hdpq = fma(fij, dot(ab[0] + i * rT, ab[1] + j * rT), hdpq);
                hdpq = fma(fji, dot(ab[0] + j * rT, ab[1] + i * rT), hdpq);
            }
            // left null space: (I - U_M U_M^T) dM V_K against P Q^T V_K
            const int r = e / K, t = e % K;   // K3 x K entries
            double v = A1[r * K + t];
            if (r < N)
                for (int b = 0; b < N; ++b) v = fma(-Um[b * N + r], EL[b * K + t], v);
            hdpq = fma(v, dot(pr[0] + r * rT, ab[1] + t * rT), hdpq);
        }
        acc = block_sum(acc, red);
        h2 = block_sum(h2, red);
        hpq = block_sum(hpq, red);
        hdh = block_sum(hdh, red);
        hdpq = block_sum(hdpq, red);
        rs = block_sum(rs, red);
        // new factors: U' = [U* Q] U_M[:, :K] = U_f (R_U^{-1} X1) + [W1 dW1] (R_G^{-1} X2)
        for (int e = tid; e < 2 * K3 * K; e += TR_THREADS) {
            const int side = e / (K3 * K), x = e % (K3 * K), i = x / K, t = x % K;
            const double* X = (side ? Vm : Um) + t * N;
            double v = 0.0;
            if (i < K) {
                for (int l = 0; l < K; ++l) v = fma(ra[side][i * K + l], X[l], v);
            } else {
                for (int l = 0; l < K; ++l) v = fma(Ri[side][(i - K) * K2 + l], X[K + l], v);
            }
            a.S[side][x] = v;
        }
        if (tid < K) a.sigma_out[tid] = sg[tid];
        if (tid == 0) {
            RelaxResult r;
            r.loss = (h2 - 2.0 * hpq + acc) / acc;
            r.dloss_dzeta = 2.0 * (hdh - hdpq) / acc;
            r.err = sqrt(rs / a.normD2);
            r.sigma1 = sg[0];
            r.sigma_r1 = sg[K];
            r.sweeps = sweeps_s;
            r.pad = 0;
            *a.result = r;
        }
    }

    static __device__ void run(const Args& a) {
        if (a.stage == 1) stage1(a);
        else stage2(a);
    }
};

template <typename T, int K> hipError_t relax_run(const RelaxArgs& a, hipStream_t s) {
    TrainPass<T> tp;
    memset(&tp, 0, sizeof(tp));
    tp.D = a.D;
    tp.ldd = a.ldd;
    tp.m = a.m;
    tp.n = a.n;
    tp.TM = a.TM;
    tp.n_ct = a.n_ct;
    tp.n_rt = a.n_rt;
    tp.zeta = a.zeta;
    tp.itau = fmin(1.0 / a.tau, DBL_MAX);
    tp.Lr = {cptr<T>(a.AL), K};
    tp.Lc = {cptr<T>(a.BL), K};
    tp.r0 = {cptr<T>(a.Uf), K};
    tp.c0 = {cptr<T>(a.Vf), K};
    tp.Rp = a.R1;
    tp.Cp = a.R2;
    tp.scal = a.Rres;
    hipLaunchKernelGGL((k_train_pass<T, T, K, TRAIN_STEP>), dim3((unsigned)(a.n_ct * a.n_rt)), dim3(TP_THREADS), 0, s,
                       tp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int K2 = 2 * K;
    const int rt = a.rt_true;
    const bool f32 = sizeof(T) == 4;
    const PanelRef F[2] = {panel_ref(a.Uf, K, K, f32), panel_ref(a.Vf, K, K, f32)};
    const PanelRef Y[2] = {panel_ref(a.RY1, K2, K2), panel_ref(a.RY2, K2, K2)};
    const PanelRef PT[2] = {panel_ref(a.P, rt, rt), panel_ref(a.Q, rt, rt)};
    const int rows[2] = {a.m, a.n}, tiles[2] = {a.n_ct, a.n_rt};
    const double* part[2] = {a.R1, a.R2};
    double* ry[2] = {a.RY1, a.RY2};
    double* out[2] = {a.Uout, a.Vout};
    StepArgs<RelaxTailArgs> base;
    memset(&base, 0, sizeof(base));
    base.gpart = a.gpartR;
    base.cnt = &a.ctrl->cnt[CNT_RELAX];
    RelaxTailArgs& t = base.tail;
    t.rt = rt;
    t.Rinv[0] = a.RUinv;
    t.Rinv[1] = a.RVinv;
    t.C = a.coef + 4 * 3 * K * K;   // after the two coefficient blocks (3K x 2K each)
    t.scal = a.Rres;
    t.tiles = a.n_tiles;
    t.normD2 = a.normD2;
    t.sigma_out = a.sigma_out;
    t.result = a.result;
    for (int side = 0; side < 2; ++side) {
        t.G1[side] = a.gram + side * RX_WMAX * RX_WMAX;
        t.G2[side] = a.gram2 + side * RX_WMAX * RX_WMAX;
        t.S[side] = a.coef + side * 2 * 3 * K * K;
        step_rows(&base.side[side], rows[side]);
    }
    StepArgs<RelaxTailArgs> s1 = base, s2 = base, s3 = base;
    s1.tail.stage = 1;
    s2.tail.stage = 2;
    for (int side = 0; side < 2; ++side) {
        double* g1 = a.gram + side * RX_WMAX * RX_WMAX;
        double* g2 = a.gram2 + side * RX_WMAX * RX_WMAX;
        step_sum(&s1.side[side], part[side], tiles[side], K2, ry[side]);
        step_gram(&s1.side[side], {F[side], PT[side]}, {Y[side], PT[side]}, g1);
        step_comb(&s2.side[side], {Y[side], F[side]}, t.S[side], K2, ry[side], K2);
        step_gram(&s2.side[side], {Y[side]}, {Y[side], PT[side]}, g2);
        step_comb(&s3.side[side], {F[side], Y[side]}, t.S[side], K, out[side], K);
    }
    if ((e = launch_step<RelaxTail<K>>(s1, s)) != hipSuccess) return e;
    if ((e = launch_step<RelaxTail<K>>(s2, s)) != hipSuccess) return e;
    return launch_step<RelaxTail<K>>(s3, s);
}

template <typename T> hipError_t relax_dispatch(const RelaxArgs& a, hipStream_t s) {
    switch (a.K) {
#define RPCA_CASE(KK) case KK: return relax_run<T, KK>(a, s);
        RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5) RPCA_CASE(6)
        RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10)
#undef RPCA_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_relax(const RelaxArgs& a, int dtype, hipStream_t s) {
    return dtype == 1 ? relax_dispatch<float>(a, s) : relax_dispatch<double>(a, s);
}

}  // namespace rpca
