// Shared definitions of librpca: workspace control block, small FP64 matrix
// area, launch constants and device helpers used by several kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace rpca {

constexpr int KMAX = 16;          // largest rank / init block handled by the kernels
constexpr int WAVE = 64;          // CDNA wavefront width
constexpr int STREAM_THREADS = 256;
constexpr int STREAM_WAVES = STREAM_THREADS / WAVE;
constexpr int STREAM_CPL = 4;     // consecutive columns owned by one lane
constexpr int STREAM_TN = WAVE * STREAM_CPL;   // columns per stream tile
constexpr int PANEL_THREADS = 256;
constexpr int GATHER_SPLIT = 8;   // adjacent lanes sharing one row in the gather kernel (<= 16)
constexpr int GATHER_THREADS = 1024;        // gather workgroup: 128 rows
constexpr int GATHER_THREADS_SMALL = 512;   // gather workgroup for small problems: 64 rows
constexpr int GATHER_SMALL_MAX_ROWS = 8192; // m + n up to which the small workgroup is used
// Threads per workgroup of the gather kernel for an m x n problem. Halving the
// rows per workgroup below m + n = 8192 spreads the small problems' partial
// sums over twice as many CUs (2-3 % faster solves at m = n = 2000-3000, 7 %
// for a batch of 2000 x 2000 instances); above, the last workgroup's sum over
// the doubled number of partials costs more than that gains.
__host__ __device__ constexpr int gather_threads_for(int64_t m, int64_t n) {
    return m + n <= GATHER_SMALL_MAX_ROWS ? GATHER_THREADS_SMALL : GATHER_THREADS;
}
constexpr int GPART_STRIDE = 2 * KMAX * KMAX;   // doubles per workgroup partial slot
// relaxed iteration (threshold training)
constexpr int RX_KMAX = 10;        // largest rank of the relaxed iteration (3r columns of a combination, at most 32)
constexpr int RX_TRUE_MAX = 16;    // largest rank of the loss's target factors
constexpr int RX_THREADS = 256;    // columns per tile of its pass over D
constexpr int RX_MAX_RT = 32;      // row tiles of that pass: 256 tiles, one per CU, at m = n = 2000
constexpr int RX_WMAX = 3 * RX_KMAX + RX_TRUE_MAX;   // widest Gram, [F Y dY P]
// panel steps of the relaxed iterations (train_panel.hpp)
constexpr int TR_THREADS = 256;
constexpr int TR_WAVES = TR_THREADS / WAVE;
constexpr int TR_ROWS = 16 * TR_WAVES;   // rows of a workgroup at a time
constexpr int TR_MAX_BLK = 64;           // workgroups per side, each looping over its rows: the last
                                         // workgroup sums the Gram partials of all of them
constexpr int TR_GE = 2048;              // entries of a Gram partial (and of a small-matrix slot)
__host__ __device__ constexpr int train_rows_per_block(int64_t rows) {
    const int64_t units = (rows + TR_ROWS - 1) / TR_ROWS;
    return (int)((units + TR_MAX_BLK - 1) / TR_MAX_BLK) * TR_ROWS;
}
__host__ __device__ constexpr size_t train_gpart_doubles(int64_t m, int64_t n) {
    return (size_t)((m + train_rows_per_block(m) - 1) / train_rows_per_block(m) +
                    (n + train_rows_per_block(n) - 1) / train_rows_per_block(n)) * TR_GE;
}
// threshold network: phi (4) -> 32 -> 32 -> 1
constexpr int MLP_IN = 4, MLP_H = 32;
constexpr int MLP_PARAMS = MLP_H * MLP_IN + MLP_H + MLP_H * MLP_H + MLP_H + MLP_H + 1;   // 1249
constexpr double MLP_K_FEAT = 15.0;   // iteration count that normalises the first feature
// sigma_{r+1} / sigma_1 enters the features clamped from below: the FP32 path
// resolves sigma_{r+1} only to about 1e-5 sigma_1, so smaller ratios are noise
constexpr double MLP_SIGMA_RATIO_FLOOR = 1e-4;

// Stages of the device-side state machine (Ctrl::stage).
enum Stage : int {
    STAGE_SIGMA_D = 0,   // init: subspace iteration on D for sigma_1(D)
    STAGE_INIT_Z = 1,    // init: subspace iteration on D - T_{zeta_-1}(D)
    STAGE_INIT_DONE = 2, // init converged; host switches to rank-r kernels
    STAGE_MAIN = 3,      // AccAltProj loop
    STAGE_FAILED = 4,    // init stopped: ||D||_F = 0 or a non-finite entry in D
};

// Which loop a kernel launch belongs to (gating of speculatively queued bodies).
enum Body : int {
    BODY_INIT = 0,   // runs only while the initial subspace iteration is in progress
    BODY_MAIN = 1,   // runs only while the AccAltProj loop has not stopped
    BODY_ANY = 2,    // always runs (single steps, tests)
};

// Counter slots for the last-workgroup-finishes pattern.
enum CounterSlot : int {
    CNT_GATHER = 0, CNT_COMPLEMENT = 1, CNT_UPDATE = 2, CNT_BASIS = 3, CNT_START = 4, CNT_RELAX = 5, CNT_CROSS = 6,
    CNT_COUNT = 8,
};

// Completion record of one queued body, written into mapped host memory by
// the body's last kernel (ring slot id & (BODY_RING - 1)); id is written last.
struct BodyRecord {
    int32_t id;          // body id given by the host (> 0)
    int32_t stage;
    int32_t done;        // loop finished
    int32_t k;
    double err;          // err of the state the body started from (loop bodies)
};
constexpr int BODY_RING = 8;

// Control block at the start of the workspace (device memory).
struct Ctrl {
    uint32_t cnt[CNT_COUNT];
    int32_t done;        // main loop finished (err < tol or k == max_iter)
    int32_t stage;
    int32_t k;           // index of the current state (L_k, S_k)
    int32_t passes;      // passes over D in the current init stage
    int32_t total_passes;
    int32_t max_iter;
    int32_t keep;        // singular triplets kept from M (p in init, r in main)
    int32_t r;
    int32_t p;
    int32_t init_max_passes;
    int32_t trim;        // 1: apply Algorithm 2 in the update kernel
    int32_t want_stop;   // 1: gather kernel applies the stopping rule
    int32_t stopped_by_tol;
    int32_t active;      // 1 while the current loop body is live (set by the gather kernel)
    int32_t jacobi_sweeps;   // sweeps of the last 2K x 2K SVD (diagnostic)
    int32_t post_update; // 1 (Gram only) or 2 (Gram and cross products): the update kernel left
                         // the sums of its partials to workgroup 0 of the next streaming pass
    double zeta;         // threshold used by the next stream pass
    double err;          // err of the current state
    double normD2;       // ||D||_F^2
    double beta, beta_init, gamma, mu, tol;
    double res_prev;     // init convergence tracking
    double sigma1_D;
    double sig1_pt, sigr1_pt;   // sigma_1 and sigma_{r+1} of the last P_T(D - S_k)
    double tol_res_a, tol_res_b;
    double resid2;       // last residual sum (sum over |x| <= zeta of x^2)
    double sigma_dead;   // relative size below which a singular triplet of M is dropped
    double max_abs_D;    // max |D_ij| (from the init passes, where L = 0)
    double err_prev;     // err_{k-1} (fallback test of the learned schedule)
    int32_t learned_on;  // 1 while zeta_{k+1} comes from the threshold network
    int32_t res_carried; // 1: the init stage continues the previous stage's iteration (res_prev is its)
    int32_t single;      // 1: D and the streamed factors are FP32
    int32_t nonfinite;   // 1: ||D||_F^2 was zero or not finite (bad input);
                         // 2: a later residual sum was not finite (bad state or breakdown)
};

// Leading entries of the err and zeta histories that a solve's last kernel
// copies into its status slot; a longer history is read with two copies.
constexpr int PUBLISH_HIST = 128;
// One per call in flight on a device (a pool in mapped, coherent host memory).
struct HostStatus {
    BodyRecord body[BODY_RING];
    Ctrl fin;                        // control block published by the call's last kernel
    double hist[2][PUBLISH_HIST];    // err_0.., zeta_0.. at the end of a solve; or the
                                     // values of a call that reports no control block
    int32_t published;               // count of the call's reports so far, written last
};

// Small FP64 matrices shared between kernels (all K x K, row-major, ld = KMAX).
struct Small {
    double RUinv[KMAX * KMAX];   // R_U^{-1}: Gram(U_f) = R_U^T R_U
    double RVinv[KMAX * KMAX];
    double Cstar[KMAX * KMAX];   // C* = R_U^{-T} U_f^T Y1 R_V^{-1}
    double C2[KMAX * KMAX];      // C2 = R_V^{-T} V_f^T Y2 R_U^{-1}  (= C*^T up to rounding)
    double E1[KMAX * KMAX];      // U_new = U_f E1 + S_U E2  (S_U = Y1 or W1)
    double E2[KMAX * KMAX];
    double F1[KMAX * KMAX];      // V_new = V_f F1 + S_V F2  (S_V = Y2 or W2)
    double F2[KMAX * KMAX];
    double RAinv[KMAX * KMAX];   // Gram(A) = R_A^T R_A (Trim output)
    double RBinv[KMAX * KMAX];
    double sigma_new[KMAX];
    double sigma_M[2 * KMAX];
    // Cross products of the rebuild factors with the bases of a streaming
    // pass: GAU = AL^T U_f, GBV = BL^T V_f (products of the stored values).
    // With Z = D - S = L + E, E = D - L - S, the pass forms E V_f and E^T U_f
    // and the gather adds L V_f = AL GBV and L^T U_f = BL GAU.
    double GAU[KMAX * KMAX];
    double GBV[KMAX * KMAX];
};

__host__ __device__ constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---------------------------------------------------------------- device --

template <typename T> struct AccOf;
template <> struct AccOf<float> { using type = float; };
template <> struct AccOf<double> { using type = double; };

// Sum of one double over the threads of a workgroup (result valid in all
// threads; fixed order). red: shared scratch of blockDim.x / 64 doubles.
__device__ inline double block_sum(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    const int w = threadIdx.x / WAVE;
    const int nw = blockDim.x / WAVE;
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < nw; ++i) s += red[i];
    __syncthreads();
    return s;
}
__device__ inline double block_sum_256(double v, double* red) { return block_sum(v, red); }

// Whether a streaming pass / gather launch of the given body executes.
__device__ inline bool body_runs(const Ctrl* c, int body) {
    if (body == BODY_INIT) return c->stage == STAGE_SIGMA_D || c->stage == STAGE_INIT_Z;
    if (body == BODY_MAIN) return c->done == 0;
    return true;
}

// Tile handled by workgroup b of a G-workgroup launch. Workgroups are handed to
// the 8 XCDs of the device in turn (b, b + 8, ... on XCD b % 8); numbering the
// tiles so that each XCD takes one contiguous run puts neighbouring tiles
// (the column tiles of a row band, which share the cache lines at their
// edges) on one XCD and its L2. A bijection of 0..G-1.
__device__ inline int xcd_tile(int b, int G) {
    constexpr int NX = 8;
    const int q = G / NX, rm = G % NX;
    const int x = b % NX, pos = b / NX;
    return (x < rm ? x * (q + 1) : rm * (q + 1) + (x - rm) * q) + pos;
}

// Loads of D, which every pass reads exactly once. NT: marked non-temporal, so
// that streaming the m x n data does not evict from the L2 what the kernels
// around the pass reuse (bases, partial sums, code). FP32 passes up to
// D_LOADS_NT_KMAX columns: a learned solve at m = n = 10^4, r = 5, took
// 1.64 ms with plain loads, 1.50 with these. Beyond, where the vector ALU work
// bounds the pass, they made it 5 % slower (r = 10), as they did FP64 passes
// (8-byte D) at every size measured (m = n = 5000: solve 2.09 -> 2.43 ms).
constexpr int D_LOADS_NT_KMAX = 6;
template <bool NT> __device__ inline float load_d(const float* p) {
    if constexpr (!NT) return *p;
    return __builtin_nontemporal_load(p);
}
template <bool NT> __device__ inline double load_d(const double* p) {
    if constexpr (!NT) return *p;
    return __builtin_nontemporal_load(p);
}

// Element-aligned 16-byte vectors: the hardware takes 16-byte accesses at any
// 4-byte address, so code using them needs no alignment of rows.
template <typename T> struct Vec16u;
template <> struct Vec16u<float> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec16u<double> { typedef double type __attribute__((ext_vector_type(2), aligned(8))); };

// Rows j .. j + R - 1 of an n x K panel into registers, zeros past the first
// nv of them. The R K values are contiguous: whole vectors when all R are there.
// (One conditional 4-byte load per value, which this replaces in the passes, held
// each workgroup back by as many dependent branches: loop pass over 10^4 x 10^4
// at K = 5 86 -> 75 us, over 25344 x 2000 at K = 2 69 -> 36 us, 5.7 TB/s.)
template <typename T, int R, int K>
__device__ __forceinline__ void load_panel_rows(const T* __restrict__ P, int j, int nv, T (&b)[R][K]) {
    constexpr int VW = 16 / (int)sizeof(T);
    static_assert((R * K) % VW == 0, "whole vectors");
    const T* p = P + (size_t)j * K;
    if (nv == R) {
#pragma unroll
        for (int v = 0; v < R * K / VW; ++v) {
            const auto x = *reinterpret_cast<const typename Vec16u<T>::type*>(p + v * VW);
#pragma unroll
            for (int q = 0; q < VW; ++q) b[(v * VW + q) / K][(v * VW + q) % K] = x[q];
        }
    } else {
#pragma unroll
        for (int s = 0; s < R; ++s)
#pragma unroll
            for (int t = 0; t < K; ++t) b[s][t] = s < nv ? p[s * K + t] : T(0);
    }
}

// p moved by off bytes (the data of another instance of a batched launch);
// a null pointer stays null.
template <typename X> __device__ inline X* shifted(X* p, int64_t off) {
    return p ? reinterpret_cast<X*>(reinterpret_cast<uintptr_t>(p) + (uintptr_t)off) : p;
}
// The same for a pointer that is never null, as plain address arithmetic
// (keeps a kernel argument in scalar registers).
template <typename X> __device__ inline X* moved(X* p, int64_t off) {
    using C = typename std::conditional<std::is_const<X>::value, const char, char>::type;
    return reinterpret_cast<X*>(reinterpret_cast<C*>(p) + off);
}

// Stores a partial result that the last workgroup of this launch reads: an
// agent-scope store, which goes through this XCD's L2 to where every XCD sees it.
__device__ inline void store_agent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Last-workgroup election: signals that this workgroup's partial results (stored
// with store_agent, by any of its threads) are there; returns true in all threads
// of the single workgroup that finished last, to which all of them are visible.
// The counter is reset by the caller. Every wave first waits until its own stores
// have completed (the workgroup barrier alone waits only for LDS operations).
// Since those stores went through to where all XCDs see them, the increment
// needs no release: that writes back the XCD's whole L2, the panel rows included,
// once for every workgroup. (A batch of 24 calls, 2000 x 2000, K = 6: 4.13 ms with
// a release, 3.50 without; one call at 25344 x 2000, K = 2: 1.86 and 1.81.) The
// last workgroup acquires, so that its loads of the partials miss its own caches.
// Results written with ordinary stores are not covered: they are for later kernels.
__device__ inline bool last_block_arrives(uint32_t* counter, int* flag_smem) {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = (prev == gridDim.x - 1) ? 1 : 0;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *flag_smem = last;
    }
    __syncthreads();
    return *flag_smem != 0;
}

}  // namespace rpca
