// Reverse mode of K unrolled relaxed iterations (training of a threshold
// schedule; not part of the paper).
//
// One relaxed body from L_k = U diag(sigma) V^T (Algorithm 1 with the hard
// threshold replaced by s(x) = x logistic((|x| - zeta) / tau)):
//   Trim (Algorithm 2): A = diag(w_U) U, B = diag(w_V) V; U~ = A R_A^{-1},
//   V~ = B R_B^{-1} (Cholesky QR);  X = D - L_k,  Z = D - s(X);
//   Y1 = Z V~, Y2 = Z^T U~, C = U~^T Y1, W1 = Y1 - U~ C = Q1 R1, W2 = Y2 - V~ V~^T Y2 = Q2 R2;
//   M = [[C, R2^T], [R1, 0]] = U_M S V_M^T;  L_{k+1} = H_r(P_T(Z)) = B_U H_r(M) B_V^T,
//   B_U = [U~ Q1], B_V = [V~ Q2]   (Section 2.1).
// The loss is sum_k w_k ||L_k - P Q^T||_F^2 / ||P Q^T||_F^2 over the iterates.
//
// Between bodies the gradient is taken with respect to L_k (the next body
// depends on the factors only through L_k and its spans), and it is never
// formed: it is Lbar_k = Zbar_k o s'(X_k) + F1 V^T + U F2^T (o the entrywise
// product), with the tangent-space matrix Zbar_k = U~ X_^T + Y_ V~^T. Body k's
// reverse step needs only Gamma_V = Lbar_{k+1} B_V and Gamma_U = Lbar_{k+1}^T B_U
// (thin), which the previous reverse step forms while it streams over D. Per
// body, with Mhat = B_U^T Gamma_V:
//   H_r:  Ybar = B_U Kc B_V^T + Gt_V Pi_V B_V^T + B_U Pi_U Gt_U^T,
//         Kc = U_M Phi(U_M^T Mhat V_M) V_M^T (Phi: the first-order coefficients
//         of the top-r singular triplets, a symmetric map), Pi_U = U_M,r U_M,r^T,
//         Pi_V = V_M,r V_M,r^T, Gt_V = Gamma_V - B_U Mhat, Gt_U = Gamma_U - B_V Mhat^T;
//   P_T:  Zbar = P_T(Ybar) = U~ X_^T + Y_ V~^T, and for the projectors
//         G_U = (Pbar_U + Pbar_U^T) U~ = (B_U Kc[:, r:] + Gt_V Pi_V[:, r:]) R2 + Z N_V,
//         G_V = (B_V Kc[r:, :]^T + Gt_U Pi_U[:, r:]) R1 + Z^T N_U,
//         N_V = (I - P_V) Ybar^T U~, N_U = (I - P_U) Ybar V~ = Y_;
//   QR:   Abar = (I - P_U) G_U R_A^{-T};  Trim: Ubar_i = w_i Abar_i - [|U_i| > c] (c/|U_i|^3)(Abar_i . U_i) U_i;
//   s:    dloss/dzeta_k = sum Zbar o X g (1 - g) / tau;  dZ/dL = s'(X) = g + |X| g (1 - g) / tau;
//   to L_k: F1 = (I - U U^T) Ubar_trim Sigma^{-1}, F2 = (I - V V^T) Vbar_trim Sigma^{-1}.
// At the first body the gradients with respect to the free factors are
// returned: Ubar_0 = (Zbar o s') V Sigma + Ubar_trim, Vbar_0 likewise,
// sigmabar_t = U_t^T (Zbar o s') V_t.
//
// Kernels: a pass over D per body and direction (recompute of Y1, Y2; then
// Z N_V, Z^T N_U, the zeta derivative and the Hadamard products with the
// previous body's bases), thin Grams summed in a fixed order, thin row
// combinations out = [panels] S with S formed by FP64 tails, and
// the row-local Trim steps. Everything but D is FP64.

#include <math.h>
#include <string.h>

#include <initializer_list>

#include "../../include/rpca.h"
#include "launch.hpp"
#include "train_panel.hpp"
#include "train_pass.hpp"
#include "wave.hpp"

namespace rpca {
namespace {

// ---- the small FP64 algebra, by the last workgroup of a panel step ------------------
//
// Small matrices are row-major unless stated; the SVD of M keeps the
// column-major layout of the Jacobi routine (vector b in entries b N .. b N + N - 1).
// The factorisations run in one wave, everything else in all threads.
enum TailMode : int {
    T_NONE = 0, T_CHOL = 1, T_C = 2, T_CHOL_M = 3, T_B2 = 4, T_ABAR = 5, T_F = 6, T_GAMMA = 7, T_NT = 8, T_OUT0 = 9
};

struct TailArgs {
    const double* in[6];
    double* out[7];
    double c;       // loss coefficient 2 w / ||P Q^T||^2 (without the division)
    int32_t rt;     // rank of the target factors
    int32_t init;   // gamma tail: the first reverse step (no H, F panels)
    int32_t mode;
};

template <int K> struct AdjTail {
    using Args = TailArgs;
    static constexpr int N = 2 * K;

    // in[0], in[1]: K x K Grams (U side, V side) -> out[0], out[1]: R^{-1};
    // out[2], out[3]: R (when given). With m (the complements' Grams): also the
    // SVD of M = [[C, R2^T], [R1, 0]], C = in[2] -> out[4] = U_M, out[5] = S, out[6] = V_M
    static __device__ __forceinline__ void chol(const Args& a, bool m) {
        __shared__ double G0[K * K], G1[K * K], R0[K * K], R1[K * K], I0[K * K], I1[K * K];
        __shared__ double Mm[N * N], Uo[N * N], Vo[N * N], sg[N];
        __shared__ JacobiLds<N> jac;
        const int tid = threadIdx.x;
        for (int e = tid; e < K * K; e += TR_THREADS) {
            G0[e] = a.in[0][e];
            G1[e] = a.in[1][e];
        }
        __syncthreads();
        if (tid < WAVE) w_chol_inv2<K>(G0, R0, I0, G1, R1, I1);
        __syncthreads();
        for (int e = tid; e < K * K; e += TR_THREADS) {
            a.out[0][e] = I0[e];
            a.out[1][e] = I1[e];
            if (a.out[2]) a.out[2][e] = R0[e];
            if (a.out[3]) a.out[3][e] = R1[e];
        }
        if (!m) return;
        // column-major: element (row, col) at col * N + row
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int col = e / N, row = e % N;
            double v = 0.0;
            if (row < K && col < K) v = a.in[2][row * K + col];
            else if (row < K) v = R1[(col - K) * K + row];
            else if (col < K) v = R0[(row - K) * K + col];
            Mm[e] = v;
        }
        __syncthreads();
        jacobi_svd<N, false>(tid / WAVE, Mm, sg, Uo, Vo, &jac);
        for (int e = tid; e < N * N; e += TR_THREADS) {
            a.out[4][e] = Uo[e];
            a.out[6][e] = Vo[e];
        }
        if (tid < N) a.out[5][tid] = sg[tid];
    }

    // in[0] = U~^T Y1, in[1] = V~^T Y2 (K x K) -> out[0] = [[I], [-C]], out[1] = [[I], [-C2]] (2K x K); out[2] = C
    static __device__ __forceinline__ void c_blocks(const Args& a) {
        for (int e = threadIdx.x; e < 2 * K * K; e += TR_THREADS) {
            const int r = e / K, c = e % K;
            const double id = (r == c) ? 1.0 : 0.0;
            a.out[0][e] = r < K ? id : -a.in[0][(r - K) * K + c];
            a.out[1][e] = r < K ? id : -a.in[1][(r - K) * K + c];
        }
        for (int e = threadIdx.x; e < K * K; e += TR_THREADS) a.out[2][e] = a.in[0][e];
    }

    // Reverse step of H_r. in[0] = Mhat = B_U^T Gamma_V (2K x 2K row-major),
    // in[1] = U_M, in[2] = S, in[3] = V_M (column-major), in[4] = R1, in[5] = R2.
    // out[0] = S_U (4K x 2K): [Y_ | GU0] = [B_U | Gamma_V] S_U;
    // out[1] = S_V (4K x 3K): [X_ | N_V | GV0] = [B_V | Gamma_U] S_V.
    static __device__ __forceinline__ void b2(const Args& a) {
        __shared__ double Mh[N * N], Um[N * N], Vm[N * N], sg[N], E[N * N], F[N * N], T1[N * N], Kc[N * N];
        __shared__ double PU[N * N], PV[N * N], A1[N * N], A2[N * N], Tn[N * K], r1[K * K], r2[K * K];
        const int tid = threadIdx.x;
        // singular vectors of negligible singular values are not defined by the
        // one-sided method: drop them (their part enters through the projector term)
        const double cut = 1e-12 * a.in[2][0];
        for (int e = tid; e < N * N; e += TR_THREADS) {
            Mh[e] = a.in[0][e];
            Um[e] = a.in[2][e / N] > cut ? a.in[1][e] : 0.0;
            Vm[e] = a.in[3][e];
        }
        for (int e = tid; e < K * K; e += TR_THREADS) {
            r1[e] = a.in[4][e];
            r2[e] = a.in[5][e];
        }
        if (tid < N) sg[tid] = a.in[2][tid];
        __syncthreads();
        // T1 = Mhat V_M (row-major), E = U_M^T T1; the projectors Pi_U, Pi_V
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int r = e / N, b = e % N;
            double v = 0.0, pu = 0.0, pv = 0.0;
            for (int c = 0; c < N; ++c) v = fma(Mh[r * N + c], Vm[b * N + c], v);
            for (int t = 0; t < K; ++t) {
                pu = fma(Um[t * N + r], Um[t * N + b], pu);
                pv = fma(Vm[t * N + r], Vm[t * N + b], pv);
            }
            T1[e] = v;
            PU[e] = pu;
            PV[e] = pv;
        }
        __syncthreads();
        // E; A1 = Mhat Pi_V, A2 = Mhat^T Pi_U (row-major N x N)
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int i = e / N, j = e % N;
            double v = 0.0, v1 = 0.0, v2 = 0.0;
            for (int l = 0; l < N; ++l) {
                v = fma(Um[i * N + l], T1[l * N + j], v);
                v1 = fma(Mh[i * N + l], PV[l * N + j], v1);
                v2 = fma(Mh[l * N + i], PU[l * N + j], v2);
            }
            E[e] = v;
            A1[e] = v1;
            A2[e] = v2;
        }
        __syncthreads();
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int i = e / N, j = e % N;
            double f = 0.0;
            if (i < K && j < K) {
                f = E[e];
            } else if (i < K) {
                const double si = sg[i], sj = sg[j];
                f = (si * si * E[i * N + j] + si * sj * E[j * N + i]) / (si * si - sj * sj);
            } else if (j < K) {
                const double si = sg[j], sj = sg[i];
                f = (si * si * E[i * N + j] + si * sj * E[j * N + i]) / (si * si - sj * sj);
            }
            F[e] = f;
        }
        for (int e = tid; e < N * K; e += TR_THREADS) {
            const int r = e / K, t = e % K;   // Tn = (I - U U^T) Mhat V_K, N x K
            double v = T1[r * N + t];
            for (int b = 0; b < N; ++b) v = fma(-Um[b * N + r], E[b * N + t], v);
            Tn[e] = v;
        }
        __syncthreads();
        // Kc = U_M F V_M^T + (I - U_M U_M^T) Mhat V_M,K V_M,K^T (the dropped left vectors)
        for (int e = tid; e < N * N; e += TR_THREADS) {   // T1 = U_M F (row-major)
            const int r = e / N, j = e % N;
            double v = 0.0;
            for (int i = 0; i < N; ++i) v = fma(Um[i * N + r], F[i * N + j], v);
            T1[e] = v;
        }
        __syncthreads();
        for (int e = tid; e < N * N; e += TR_THREADS) {
            const int r = e / N, c = e % N;
            double v = 0.0;
            for (int j = 0; j < N; ++j) v = fma(T1[r * N + j], Vm[j * N + c], v);
            for (int t = 0; t < K; ++t) v = fma(Tn[r * K + t], Vm[t * N + c], v);
            Kc[e] = v;
        }
        __syncthreads();
        // S_U rows 0..N-1 (B_U): [Khat - Mhat Pi_V[:, :K] | (Kc[:, K:] - Mhat Pi_V[:, K:]) R2];
        //     rows N..2N-1 (Gamma_V): [Pi_V[:, :K] | Pi_V[:, K:] R2]
        for (int e = tid; e < 2 * N * N; e += TR_THREADS) {
            const int r = e / N, c = e % N;
            double v = 0.0;
            if (r < N) {
                if (c < K) {
                    v = (r >= K ? Kc[r * N + c] : 0.0) - A1[r * N + c];
                } else {
                    for (int l = 0; l < K; ++l) v = fma(Kc[r * N + K + l] - A1[r * N + K + l], r2[l * K + (c - K)], v);
                }
            } else {
                const int rr = r - N;
                if (c < K) {
                    v = PV[rr * N + c];
                } else {
                    for (int l = 0; l < K; ++l) v = fma(PV[rr * N + K + l], r2[l * K + (c - K)], v);
                }
            }
            a.out[0][e] = v;
        }
        // S_V rows 0..N-1 (B_V): [Kc[:K, :]^T - Mhat^T Pi_U[:, :K] | [0; Kc[:K, K:]^T] - Mhat^T Pi_U[:, :K] |
        //                         (Kc[K:, :]^T - Mhat^T Pi_U[:, K:]) R1];
        //     rows N..2N-1 (Gamma_U): [Pi_U[:, :K] | Pi_U[:, :K] | Pi_U[:, K:] R1]
        for (int e = tid; e < 2 * N * 3 * K; e += TR_THREADS) {
            const int r = e / (3 * K), c = e % (3 * K);
            double v = 0.0;
            if (r < N) {
                if (c < K) {
                    v = Kc[c * N + r] - A2[r * N + c];
                } else if (c < 2 * K) {
                    v = (r >= K ? Kc[(c - K) * N + r] : 0.0) - A2[r * N + (c - K)];
                } else {
                    for (int l = 0; l < K; ++l)
                        v = fma(Kc[(K + l) * N + r] - A2[r * N + K + l], r1[l * K + (c - 2 * K)], v);
                }
            } else {
                const int rr = r - N;
                if (c < 2 * K) {
                    v = PU[rr * N + (c % K)];
                } else {
                    for (int l = 0; l < K; ++l) v = fma(PU[rr * N + K + l], r1[l * K + (c - 2 * K)], v);
                }
            }
            a.out[1][e] = v;
        }
    }

    // in[0] = U~^T G_U, in[1] = V~^T G_V, in[2] = R_A^{-1}, in[3] = R_B^{-1} ->
    // out[0] = [[R_A^{-T}], [-(U~^T G_U) R_A^{-T}]] (2K x K) for Abar = [G_U | U~] S; out[1] likewise
    static __device__ __forceinline__ void abar(const Args& a) {
        for (int x = threadIdx.x; x < 4 * K * K; x += TR_THREADS) {
            const int side = x / (2 * K * K), e = x % (2 * K * K);
            const double* G = a.in[side];
            const double* Ri = a.in[2 + side];
            const int r = e / K, c = e % K;
            double v = 0.0;
            if (r < K) {
                v = Ri[c * K + r];
            } else {
                for (int l = 0; l < K; ++l) v = fma(G[(r - K) * K + l], Ri[c * K + l], v);
                v = -v;
            }
            a.out[side][e] = v;
        }
    }

    // in[0] = U^T Ubar_trim, in[1] = V^T Vbar_trim, in[2] = sigma ->
    // out[0] = [[Sigma^{-1}], [-(U^T Ubar_trim) Sigma^{-1}]] (2K x K) for F1 = [Ubar_trim | U] S; out[1] likewise
    static __device__ __forceinline__ void f_blocks(const Args& a) {
        for (int x = threadIdx.x; x < 4 * K * K; x += TR_THREADS) {
            const int side = x / (2 * K * K), e = x % (2 * K * K);
            const int r = e / K, c = e % K;
            const double is = 1.0 / a.in[2][c];
            a.out[side][e] = r < K ? (r == c ? is : 0.0) : -a.in[side][(r - K) * K + c] * is;
        }
    }

    // Gamma for the previous body. in[0] = [U_k | F1 | P]^T B_U' ((2K + rt) x 2K),
    // in[1] = [V_k | F2 | Q]^T B_V', in[2] = sigma_k, in[3] = ||P Q^T||^2 (one value).
    // out[0] = S for Gamma_V' = [H_V | F1 | U_k | P] S (rows 2K + K + K + rt, 2K columns),
    // out[1] = S for Gamma_U' = [H_U | F2 | V_k | Q] S.
    // init: the first reverse step: Gamma_V = [U_K | P] S (rows K + rt) from
    // in[1] = [V_K | Q]^T B_V; Gamma_U = [V_K | Q] S from in[0] = [U_K | P]^T B_U.
    static __device__ __forceinline__ void gamma(const Args& a) {
        const int rt = a.rt;
        const double c = a.c / a.in[3][0];
        for (int side = 0; side < 2; ++side) {
            // Gamma_V (side 0) takes the V-side Gram, Gamma_U (side 1) the U-side one
            const double* G = a.in[side == 0 ? 1 : 0];
            // G rows: [X_k (K) | F (K) | T (rt)] (init: [X_k (K) | T (rt)])
            const int offT = a.init ? K : 2 * K;
            const int rows = a.init ? K + rt : 2 * N + rt;
            for (int e = threadIdx.x; e < rows * N; e += TR_THREADS) {
                const int r = e / N, col = e % N;
                double v;
                if (a.init) {
                    v = r < K ? c * a.in[2][r] * G[r * N + col] : -c * G[(offT + r - K) * N + col];
                } else if (r < N) {
                    v = (r == col) ? 1.0 : 0.0;
                } else if (r < N + K) {
                    v = G[(r - N) * N + col];                                   // X_k^T B'
                } else if (r < N + 2 * K) {
                    const int t = r - N - K;
                    v = G[(K + t) * N + col] + c * a.in[2][t] * G[t * N + col];  // F^T B' + c Sigma X_k^T B'
                } else {
                    v = -c * G[(offT + r - N - 2 * K) * N + col];
                }
                a.out[side][e] = v;
            }
        }
    }

    // in[0] = P^T P, in[1] = Q^T Q (rt x rt) -> out[0][0] = ||P Q^T||_F^2
    static __device__ __forceinline__ void nt(const Args& a) {
        __shared__ double red[TR_WAVES];
        double v = 0.0;
        for (int e = threadIdx.x; e < a.rt * a.rt; e += TR_THREADS) v = fma(a.in[0][e], a.in[1][e], v);
        v = block_sum(v, red);
        if (threadIdx.x == 0) a.out[0][0] = v;
    }

    // in[0] = U_0^T ((Zbar o s') V_0) (K x K), in[1] = sigma_0 ->
    // out[0][t] = sigmabar_t = in[0][t][t]; out[1] = [[Sigma], [I]] (2K x K)
    static __device__ __forceinline__ void out0(const Args& a) {
        if (threadIdx.x < K) a.out[0][threadIdx.x] = a.in[0][threadIdx.x * K + threadIdx.x];
        for (int e = threadIdx.x; e < 2 * K * K; e += TR_THREADS) {
            const int r = e / K, c = e % K;
            a.out[1][e] = r < K ? (r == c ? a.in[1][c] : 0.0) : ((r - K) == c ? 1.0 : 0.0);
        }
    }

    static __device__ void run(const Args& a) {
        switch (a.mode) {
            case T_CHOL: chol(a, false); break;
            case T_C: c_blocks(a); break;
            case T_CHOL_M: chol(a, true); break;
            case T_B2: b2(a); break;
            case T_ABAR: abar(a); break;
            case T_F: f_blocks(a); break;
            case T_GAMMA: gamma(a); break;
            case T_NT: nt(a); break;
            case T_OUT0: out0(a); break;
            default: break;
        }
    }
};

__global__ void k_adj_zero(uint32_t* p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// ---- host side ------------------------------------------------------------------------

using Step = StepArgs<TailArgs>;

struct Host {
    const AdjointProblem& P;
    const AdjointBufs& B;
    hipStream_t s;
    int K, m, n;

    // small-matrix slot i (TR_GE doubles each)
    double* sm(int i) const { return B.small + (size_t)i * TR_GE; }

    Step step(int mode = T_NONE) const {
        Step a;
        memset(&a, 0, sizeof(a));
        step_rows(&a.side[0], m);
        step_rows(&a.side[1], n);
        a.gpart = B.gpart;
        a.cnt = B.cnt;
        a.tail.mode = mode;
        a.tail.rt = P.rt;
        return a;
    }

    hipError_t run(const Step& a) const {
        switch (K) {
#define RPCA_CASE(KK) case KK: return launch_step<AdjTail<KK>>(a, s);
            RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5)
            RPCA_CASE(6) RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10)
#undef RPCA_CASE
            default: return hipErrorInvalidValue;
        }
    }

    template <typename T>
    hipError_t stream_t(const TrainPass<double>& a, bool bwd) const {
        const dim3 grid((unsigned)(a.n_ct * a.n_rt)), block(TP_THREADS);
        switch (K) {
#define RPCA_CASE(KK)                                                                                             \
    case KK:                                                                                                      \
        if (bwd) hipLaunchKernelGGL((k_train_pass<T, double, KK, TRAIN_REVERSE>), grid, block, 0, s, a);         \
        else hipLaunchKernelGGL((k_train_pass<T, double, KK, TRAIN_RECOMPUTE>), grid, block, 0, s, a);            \
        break;
            RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5)
            RPCA_CASE(6) RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10)
#undef RPCA_CASE
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }

    // one pass over D at checkpoint k (tile partials in B.Rp, B.Cp)
    hipError_t pass(int k, bool bwd, TrainPass<double> a) const {
        a.D = P.D;
        a.ldd = P.ldd;
        a.m = m;
        a.n = n;
        a.TM = P.TM;
        a.n_ct = P.n_ct;
        a.n_rt = P.n_rt;
        a.Lr = {P.U[k], K};
        a.Lc = {P.V[k], K};
        a.sig = P.sigma[k];
        a.zeta = P.zeta[k];
        a.itau = fmin(1.0 / P.tau[k], DBL_MAX);
        a.Rp = B.Rp;
        a.Cp = B.Cp;
        a.scal = B.scal;
        return P.dtype == 1 ? stream_t<float>(a, bwd) : stream_t<double>(a, bwd);
    }

    void trim(Step* a, int k, int post) const {
        const double* X[2] = {P.U[k], P.V[k]};
        const double c[2] = {P.cU, P.cV};
        for (int side = 0; side < 2; ++side) {
            a->side[side].comb.post = post;
            a->side[side].comb.K = K;
            a->side[side].comb.X = X[side];
            a->side[side].comb.c = c[side];
        }
    }

    // Forward recompute of body k into slot sl: trim, bases, Y1/Y2, complements,
    // B_U = [U~ Q1], B_V = [V~ Q2], R1, R2 and the SVD of M.
    hipError_t forward(int k, int sl) const {
        const AdjointBufs::Slot& S = B.slot[sl];
        const int N = 2 * K;
        const PanelRef A[2] = {panel_ref(S.Am, K, K), panel_ref(S.Bm, K, K)};
        const PanelRef T[2] = {panel_ref(S.BU, N, K), panel_ref(S.BV, N, K)};   // U~, V~
        const PanelRef Y[2] = {panel_ref(B.Y1, K, K), panel_ref(B.Y2, K, K)};
        const PanelRef W[2] = {panel_ref(B.W1, K, K), panel_ref(B.W2, K, K)};
        double* am[2] = {S.Am, S.Bm};
        double* bt[2] = {S.BU, S.BV};
        double* yy[2] = {B.Y1, B.Y2};
        double* ww[2] = {B.W1, B.W2};
        const double* rab[2] = {S.RAinv, S.RBinv};
        const double* r12[2] = {S.R1inv, S.R2inv};
        const double* part[2] = {B.Rp, B.Cp};
        const int tiles[2] = {P.n_ct, P.n_rt};
        hipError_t e;
        // A = Trim(U), its Gram and R_A
        Step a = step(T_CHOL);
        trim(&a, k, POST_TRIM);
        for (int side = 0; side < 2; ++side) {
            step_comb(&a.side[side], {}, nullptr, K, am[side], K);
            step_gram(&a.side[side], {A[side]}, {A[side]}, sm(side));
            a.tail.in[side] = sm(side);
        }
        a.tail.out[0] = S.RAinv;
        a.tail.out[1] = S.RBinv;
        if ((e = run(a)) != hipSuccess) return e;
        // U~ = A R_A^{-1} into the first K columns of B_U (row stride 2K)
        a = step();
        for (int side = 0; side < 2; ++side) step_comb(&a.side[side], {A[side]}, rab[side], K, bt[side], N);
        if ((e = run(a)) != hipSuccess) return e;
        // Y1 = Z V~, Y2 = Z^T U~; C = U~^T Y1
        TrainPass<double> tp;
        memset(&tp, 0, sizeof(tp));
        tp.c0 = {S.BV, N};
        tp.r0 = {S.BU, N};
        if ((e = pass(k, false, tp)) != hipSuccess) return e;
        a = step(T_C);
        for (int side = 0; side < 2; ++side) {
            step_sum(&a.side[side], part[side], tiles[side], K, yy[side]);
            step_gram(&a.side[side], {T[side]}, {Y[side]}, sm(2 + side));
            a.tail.in[side] = sm(2 + side);
            a.tail.out[side] = sm(4 + side);
        }
        a.tail.out[2] = S.C;
        if ((e = run(a)) != hipSuccess) return e;
        // W1 = Y1 - U~ C, W2 = Y2 - V~ (V~^T Y2), R1, R2 and the SVD of M
        a = step(T_CHOL_M);
        for (int side = 0; side < 2; ++side) {
            step_comb(&a.side[side], {Y[side], T[side]}, sm(4 + side), K, ww[side], K);
            step_gram(&a.side[side], {W[side]}, {W[side]}, sm(6 + side));
            a.tail.in[side] = sm(6 + side);
        }
        a.tail.in[2] = S.C;
        a.tail.out[0] = S.R1inv;
        a.tail.out[1] = S.R2inv;
        a.tail.out[2] = S.R1;
        a.tail.out[3] = S.R2;
        a.tail.out[4] = S.UM;
        a.tail.out[5] = S.SM;
        a.tail.out[6] = S.VM;
        if ((e = run(a)) != hipSuccess) return e;
        // Q1 = W1 R1^{-1} into the last K columns of B_U, Q2 likewise
        a = step();
        for (int side = 0; side < 2; ++side) step_comb(&a.side[side], {W[side]}, r12[side], K, bt[side] + K, N);
        return run(a);
    }

    // Gamma_V, Gamma_U from `in` panels and the coefficients sm(4), sm(5), then
    // Mhat = B_U^T Gamma_V of the body in slot sl and the reverse step of H_r
    hipError_t gamma_and_b2(std::initializer_list<PanelRef> inU, std::initializer_list<PanelRef> inV, int sl) const {
        const AdjointBufs::Slot& S = B.slot[sl];
        const int N = 2 * K;
        Step a = step(T_B2);
        step_comb(&a.side[0], inU, sm(4), N, B.GammaV, N);
        step_comb(&a.side[1], inV, sm(5), N, B.GammaU, N);
        step_gram(&a.side[0], {panel_ref(S.BU, N, N)}, {panel_ref(B.GammaV, N, N)}, sm(0));
        const double* in[6] = {sm(0), S.UM, S.SM, S.VM, S.R1, S.R2};
        for (int i = 0; i < 6; ++i) a.tail.in[i] = in[i];
        a.tail.out[0] = sm(1);
        a.tail.out[1] = sm(2);
        return run(a);
    }
};

}  // namespace

size_t adjoint_ws_bytes(int64_t m, int64_t n, int K, int n_ct, int n_rt) {
    AdjointBufs b;
    (void)adjoint_carve(reinterpret_cast<void*>(uintptr_t(256)), m, n, K, n_ct, n_rt, &b);
    return (size_t)(b.end - reinterpret_cast<char*>(uintptr_t(256)));
}

hipError_t adjoint_carve(void* base, int64_t m, int64_t n, int K, int n_ct, int n_rt, AdjointBufs* b) {
    char* p = static_cast<char*>(base);
    auto take = [&](size_t count) {
        double* r = reinterpret_cast<double*>(p);
        p += ((count * sizeof(double) + 255) / 256) * 256;
        return r;
    };
    const int N = 2 * K;
    const size_t W = 3 * (size_t)K;
    for (int sl = 0; sl < 2; ++sl) {
        AdjointBufs::Slot& S = b->slot[sl];
        S.Am = take(m * K);
        S.BU = take(m * N);
        S.Bm = take(n * K);
        S.BV = take(n * N);
        S.RAinv = take(TR_GE);
        S.RBinv = take(TR_GE);
        S.C = take(TR_GE);
        S.R1 = take(TR_GE);
        S.R2 = take(TR_GE);
        S.R1inv = take(TR_GE);
        S.R2inv = take(TR_GE);
        S.UM = take(TR_GE);
        S.SM = take(TR_GE);
        S.VM = take(TR_GE);
    }
    b->Y1 = take(m * K);
    b->W1 = take(m * K);
    b->GammaV = take(m * N);
    b->YG = take(m * N);
    b->SR = take(m * W);
    b->GU = take(m * K);
    b->Utrim = take(m * K);
    b->F1 = take(m * K);
    b->Y2 = take(n * K);
    b->W2 = take(n * K);
    b->GammaU = take(n * N);
    b->XG = take(n * 3 * K);
    b->SC = take(n * W);
    b->GV = take(n * K);
    b->Vtrim = take(n * K);
    b->F2 = take(n * K);
    b->Rp = take((size_t)n_ct * m * W);
    b->Cp = take((size_t)n_rt * n * W);
    b->scal = take(2 * (size_t)n_ct * n_rt);
    b->gpart = take(train_gpart_doubles(m, n));
    b->small = take(16 * (size_t)TR_GE);
    b->zbar = take(RPCA_MAX_UNROLL);
    b->cnt = reinterpret_cast<uint32_t*>(take(32));   // 64 counters
    b->end = p;
    return hipSuccess;
}

hipError_t adjoint_run(const AdjointProblem& P, const AdjointBufs& B, hipStream_t s) {
    Host h{P, B, s, P.K, (int)P.m, (int)P.n};
    const int K = P.K, N = 2 * K, Kt = P.Kt, rt = P.rt;
    hipLaunchKernelGGL(k_adj_zero, dim3(1), dim3(64), 0, s, B.cnt, 64);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const PanelRef PT[2] = {panel_ref(P.P, rt, rt), panel_ref(P.Q, rt, rt)};
    double* nt = h.sm(12);
    // ||P Q^T||^2
    Step a = h.step(T_NT);
    for (int side = 0; side < 2; ++side) {
        step_gram(&a.side[side], {PT[side]}, {PT[side]}, h.sm(10 + side));
        a.tail.in[side] = h.sm(10 + side);
    }
    a.tail.out[0] = nt;
    if ((e = h.run(a)) != hipSuccess) return e;
    // body Kt - 1 forward, then Gamma from the loss term of L_Kt
    if ((e = h.forward(Kt - 1, (Kt - 1) & 1)) != hipSuccess) return e;
    {
        const AdjointBufs::Slot& S = B.slot[(Kt - 1) & 1];
        const PanelRef X[2] = {panel_ref(P.U[Kt], K, K), panel_ref(P.V[Kt], K, K)};
        const PanelRef Bs[2] = {panel_ref(S.BU, N, N), panel_ref(S.BV, N, N)};
        a = h.step(T_GAMMA);
        for (int side = 0; side < 2; ++side) {
            step_gram(&a.side[side], {X[side], PT[side]}, {Bs[side]}, h.sm(13 + side));
            a.tail.in[side] = h.sm(13 + side);
            a.tail.out[side] = h.sm(4 + side);
        }
        a.tail.in[2] = P.sigma[Kt];
        a.tail.in[3] = nt;
        a.tail.c = 2.0 * P.weight[Kt - 1];
        a.tail.init = 1;
        if ((e = h.run(a)) != hipSuccess) return e;
        if ((e = h.gamma_and_b2({X[0], PT[0]}, {X[1], PT[1]}, (Kt - 1) & 1)) != hipSuccess) return e;
    }
    double* ga[2] = {B.GU, B.GV};
    double* tr[2] = {B.Utrim, B.Vtrim};
    double* ff[2] = {B.F1, B.F2};
    for (int k = Kt - 1; k >= 0; --k) {
        const int sl = k & 1;
        const AdjointBufs::Slot& S = B.slot[sl];
        const AdjointBufs::Slot& Sp = B.slot[sl ^ 1];
        const PanelRef X[2] = {panel_ref(P.U[k], K, K), panel_ref(P.V[k], K, K)};
        const PanelRef T[2] = {panel_ref(S.BU, N, K), panel_ref(S.BV, N, K)};   // U~, V~
        const PanelRef G[2] = {panel_ref(B.GU, K, K), panel_ref(B.GV, K, K)};
        const PanelRef Tr[2] = {panel_ref(B.Utrim, K, K), panel_ref(B.Vtrim, K, K)};
        // [Y_ | GU0] and [X_ | N_V | GV0]
        a = h.step();
        step_comb(&a.side[0], {panel_ref(S.BU, N, N), panel_ref(B.GammaV, N, N)}, h.sm(1), N, B.YG, N);
        step_comb(&a.side[1], {panel_ref(S.BV, N, N), panel_ref(B.GammaU, N, N)}, h.sm(2), 3 * K, B.XG, 3 * K);
        if ((e = h.run(a)) != hipSuccess) return e;
        // the previous body's bases (its forward recompute) for the Hadamard products
        if (k >= 1 && (e = h.forward(k - 1, sl ^ 1)) != hipSuccess) return e;
        // pass over D at L_k: Z N_V | h B_V', Z^T N_U | h B_U', dloss/dzeta_k
        TrainPass<double> tp;
        memset(&tp, 0, sizeof(tp));
        tp.c0 = {B.XG + K, 3 * K};               // N_V
        tp.r0 = {B.YG, N};                       // N_U = Y_
        if (k >= 1) {
            tp.hw = N;
            tp.c1 = {Sp.BV, N};
            tp.r1 = {Sp.BU, N};
        } else {
            tp.hw = K;
            tp.c1 = {P.V[0], K};
            tp.r1 = {P.U[0], K};
        }
        tp.Uz = {S.BU, N};
        tp.Vz = {S.BV, N};
        tp.Xz = {B.XG, 3 * K};
        tp.Yz = {B.YG, N};
        const int W = K + tp.hw;
        if ((e = h.pass(k, true, tp)) != hipSuccess) return e;
        // tile sums; G_U = GU0 + Z N_V, G_V = GV0 + Z^T N_U; U~^T G_U, V~^T G_V
        a = h.step(T_ABAR);
        step_sum(&a.side[0], B.Rp, P.n_ct, W, B.SR);
        step_sum(&a.side[1], B.Cp, P.n_rt, W, B.SC);
        a.side[0].sum.add = panel_ref(B.YG + K, N, K);
        a.side[1].sum.add = panel_ref(B.XG + 2 * K, 3 * K, K);
        a.scal = B.scal;
        a.scal_out = P.zeta_bar_dev + k;
        a.tiles = P.n_ct * P.n_rt;
        for (int side = 0; side < 2; ++side) {
            a.side[side].sum.out2 = ga[side];
            step_gram(&a.side[side], {T[side]}, {G[side]}, h.sm(6 + side));
            a.tail.in[side] = h.sm(6 + side);
            a.tail.out[side] = h.sm(8 + side);
        }
        a.tail.in[2] = S.RAinv;
        a.tail.in[3] = S.RBinv;
        if ((e = h.run(a)) != hipSuccess) return e;
        // Abar = (G_U - U~ (U~^T G_U)) R_A^{-T}, Bbar likewise, and Trim reversed
        a = h.step(k == 0 ? T_OUT0 : T_F);
        h.trim(&a, k, POST_TRIM_REVERSE);
        for (int side = 0; side < 2; ++side)
            step_comb(&a.side[side], {G[side], T[side]}, h.sm(8 + side), K, tr[side], K);
        if (k == 0) {
            // gradients of the free factors of L_0
            const PanelRef H[2] = {panel_ref(B.SR + K, W, K), panel_ref(B.SC + K, W, K)};
            step_gram(&a.side[0], {X[0]}, {H[0]}, h.sm(6));
            a.tail.in[0] = h.sm(6);
            a.tail.in[1] = P.sigma[0];
            a.tail.out[0] = P.sigma_bar;
            a.tail.out[1] = h.sm(7);
            if ((e = h.run(a)) != hipSuccess) return e;
            a = h.step();
            step_comb(&a.side[0], {H[0], Tr[0]}, h.sm(7), K, P.U_bar, K);
            step_comb(&a.side[1], {H[1], Tr[1]}, h.sm(7), K, P.V_bar, K);
            return h.run(a);
        }
        // to L_k: F1 = (I - U U^T) Ubar_trim Sigma^{-1}, F2 likewise
        for (int side = 0; side < 2; ++side) {
            step_gram(&a.side[side], {X[side]}, {Tr[side]}, h.sm(10 + side));
            a.tail.in[side] = h.sm(10 + side);
            a.tail.out[side] = h.sm(6 + side);
        }
        a.tail.in[2] = P.sigma[k];
        if ((e = h.run(a)) != hipSuccess) return e;
        // Gamma for body k - 1: Lbar_k = Zbar o s'(X_k) + F1 V^T + U F2^T + c_k (L_k - P Q^T)
        const PanelRef Fp[2] = {panel_ref(B.F1, K, K), panel_ref(B.F2, K, K)};
        const PanelRef Bp[2] = {panel_ref(Sp.BU, N, N), panel_ref(Sp.BV, N, N)};
        a = h.step(T_GAMMA);
        for (int side = 0; side < 2; ++side) {
            step_comb(&a.side[side], {Tr[side], X[side]}, h.sm(6 + side), K, ff[side], K);
            step_gram(&a.side[side], {X[side], Fp[side], PT[side]}, {Bp[side]}, h.sm(13 + side));
            a.tail.in[side] = h.sm(13 + side);
            a.tail.out[side] = h.sm(4 + side);
        }
        a.tail.in[2] = P.sigma[k];
        a.tail.in[3] = nt;
        a.tail.c = 2.0 * P.weight[k - 1];
        if ((e = h.run(a)) != hipSuccess) return e;
        if ((e = h.gamma_and_b2({panel_ref(B.SR + K, W, N), Fp[0], X[0], PT[0]},
                                {panel_ref(B.SC + K, W, N), Fp[1], X[1], PT[1]}, sl ^ 1)) != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace rpca
