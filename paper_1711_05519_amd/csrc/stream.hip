// The streaming pass over D: the only kernels of an iteration that touch the
// m x n data. One read of D computes, for the current iterate L = AL BL^T and
// threshold zeta (Section 2.1 and Algorithm 1):
//   x = D - L,  S = T_zeta(x)  (never stored),  E = D - L - S  (x where |x| <= zeta),
//   resid = sum of E_ij^2                        (numerator of err^2, Section 3)
//   E Vf,  E^T Uf
// The tangent products of the fast H_r(P_T(.)) update are Y1 = Z Vf and
// Y2 = Z^T Uf with Z = D - S = L + E; their rank-K part L Vf = AL (BL^T Vf) and
// L^T Uf = BL (AL^T Uf) is added by the gather from the factors (exactly, in
// FP64), so the pass accumulates only E, whose size is that of the residual:
// the rounding of the accumulation scales with err_k instead of with |D|. The
// threshold of iteration k and the products of iteration k+1 share one pass;
// L is rebuilt tile by tile in registers and never written.
//
// Layout: a workgroup of 4 waves owns a tile of TM rows x 256 columns. Each lane
// owns 4 consecutive columns (one 16-byte load per row for FP32) and keeps the
// matching rows of BL and Vf in registers; the 4 waves walk interleaved rows.
// Row data (AL, Uf) are wave-uniform and come through scalar loads. E^T Uf then
// accumulates per lane with no communication; the per-row sums of E Vf are
// reduced across the 64 lanes in batches with a reduce-scatter built from
// v_permlane32_swap, v_permlane16_swap and DPP moves, which leaves one finished
// sum per lane. Tile partials go to P1/P2 and are summed in FP64 by the gather
// kernel in a fixed order, so results are bitwise reproducible.
#include "launch.hpp"
#include "wave.hpp"

namespace rpca {
namespace {

template <typename T> __device__ inline T zero() { return T(0); }

// ---- cross-lane moves on 32/64-bit values ----------------------------------

__device__ inline void swap32(float& a, float& b) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ inline void swap16(float& a, float& b) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ inline void swap32(double& a, double& b) {
    uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
    auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    a = __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0]));
    b = __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ inline void swap16(double& a, double& b) {
    uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
    auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    a = __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0]));
    b = __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}

template <int CTRL> __device__ inline float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ inline double dpp(double x) {
    int64_t u = __double_as_longlong(x);
    int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// DPP controls: row_ror:8 pairs lane l with l^8; row_half_mirror with l^7;
// quad_perm[2,3,0,1] with l^2; quad_perm[1,0,3,2] with l^1.
constexpr int DPP_ROR8 = 0x128;
constexpr int DPP_HALF_MIRROR = 0x141;
constexpr int DPP_QP_2301 = 0x4E;
constexpr int DPP_QP_1032 = 0xB1;

// One level of the reduce-scatter: N values per lane -> ceil(N/2) values per
// lane. Lanes whose level bit is clear keep family 2k, the others family 2k+1.
template <int N, typename T>
__device__ inline void level_swap32(T (&x)[N], T (&y)[(N + 1) / 2]) {
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        T a = x[2 * k], b = x[2 * k + 1];
        swap32(a, b);
        y[k] = a + b;
    }
    if constexpr (N & 1) {
        T a = x[N - 1], b = zero<T>();
        swap32(a, b);
        y[N / 2] = a + b;
    }
}
template <int N, typename T>
__device__ inline void level_swap16(T (&x)[N], T (&y)[(N + 1) / 2]) {
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        T a = x[2 * k], b = x[2 * k + 1];
        swap16(a, b);
        y[k] = a + b;
    }
    if constexpr (N & 1) {
        T a = x[N - 1], b = zero<T>();
        swap16(a, b);
        y[N / 2] = a + b;
    }
}
template <int CTRL, int BIT, int N, typename T>
__device__ inline void level_dpp(T (&x)[N], T (&y)[(N + 1) / 2], int lane) {
    const bool hi = (lane >> BIT) & 1;
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        T a = x[2 * k], b = x[2 * k + 1];
        T keep = hi ? b : a;
        T send = hi ? a : b;
        y[k] = keep + dpp<CTRL>(send);
    }
    if constexpr (N & 1) y[N / 2] = x[N - 1] + dpp<CTRL>(x[N - 1]);
}

// Sums each of the V values over the 64 lanes. On return lane l holds the
// total of value index bitrev6(l) (valid when that index is < V).
template <int V, typename T>
__device__ inline T reduce_scatter64(T (&x)[V], int lane) {
    static_assert(V >= 1 && V <= 64, "reduce_scatter64 handles at most 64 values");
    constexpr int V1 = (V + 1) / 2, V2 = (V1 + 1) / 2, V3 = (V2 + 1) / 2, V4 = (V3 + 1) / 2,
                  V5 = (V4 + 1) / 2, V6 = (V5 + 1) / 2;
    static_assert(V6 == 1, "levels");
    T y1[V1], y2[V2], y3[V3], y4[V4], y5[V5], y6[V6];
    level_swap32<V>(x, y1);
    level_swap16<V1>(y1, y2);
    level_dpp<DPP_ROR8, 3, V2>(y2, y3, lane);
    level_dpp<DPP_HALF_MIRROR, 2, V3>(y3, y4, lane);
    level_dpp<DPP_QP_2301, 1, V4>(y4, y5, lane);
    level_dpp<DPP_QP_1032, 0, V5>(y5, y6, lane);
    return y6[0];
}

__device__ inline int bitrev6(int l) {
    return ((l & 1) << 5) | ((l & 2) << 3) | ((l & 4) << 1) | ((l & 8) >> 1) | ((l & 16) >> 3) |
           ((l & 32) >> 5);
}

// ---- loads of 4 consecutive elements -----------------------------------------

// Four consecutive elements of a row of D, zeros past the first nvalid.
template <bool NT, typename T>
__device__ inline void load4(const T* __restrict__ p, int nvalid, T (&d)[4]) {
    constexpr int VW = 16 / (int)sizeof(T);
    typedef typename Vec16u<T>::type VecT;
    if (nvalid == 4) {
#pragma unroll
        for (int v = 0; v < 4 / VW; ++v) {
            const VecT* q = reinterpret_cast<const VecT*>(p + v * VW);
            const VecT x = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
            for (int u = 0; u < VW; ++u) d[v * VW + u] = x[u];
        }
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] = s < nvalid ? load_d<NT>(p + s) : T(0);
    }
}

template <typename T, int K, bool REBUILD> struct StreamCfg {
    // Rows per batch per wave. The batch's wave-uniform row data (2K values of
    // AL and Uf per row) live in scalar registers. The per-element cost of the
    // reduce-scatter depends on NB * K only weakly, while the registers of the
    // two batches in flight set the occupancy. Measured over NB * K ~ 4 .. 48,
    // whole solves: up to K = 5, 16 (4 waves per SIMD at K = 3 .. 5) is the best
    // (10^4 x 10^4, K = 5 and 6 in turn: 1657, 1652, 1621, 1598, 1597, 1818 us at 4, 8,
    // 12, 16, 24, 32); from K = 6 on, where 16 is one or two rows, 24 hides more of
    // the latency than the wave it costs (24 instances of 2000 x 2000, K = 6 and 7:
    // 4.35 -> 4.22 ms; 2 10^4 x 2 10^4, initialisation at K = 11: 10.72 -> 10.45 ms).
    // A pass over 10^4 x 10^4 with 16 and 24, loop: K = 6 91 94, 7 102 110, 8 129 124, 9
    // 139 130, 10 150 142, 11 157 180, 12 208 195 us; initialisation: 6 95 93, 7 97 99, 8 108
    // 98, 9 111 104, 10 116 110, 11 128 115, 12 142 141; over 2999 x 1777 24 is as fast or up
    // to 10 % faster at every K; from K = 13 on both are one row. So 24 but for the loop at
    // K = 11 (163 VGPRs and three waves with 16, 183 and two with 24; 2 10^4 x 2 10^4 595
    // and 717 us).
    // FP64 keeps 16 words: 24 and 32 were within the spread.
    static constexpr int WORDS = (int)(sizeof(T) / 4);
    static constexpr bool DEEP = WORDS == 1 && K >= 6 && !(REBUILD && K == 11);
    static constexpr int NB0 = (DEEP ? 24 : 16) / (K * WORDS);
    static constexpr int NB = NB0 < 1 ? 1 : (NB0 > 8 ? 8 : NB0);
};

// Loads rows i0, i0 + 4, ... of the wave's 4 columns.
template <typename T, int K, bool REBUILD, bool FULL, bool CHECK>
__device__ __forceinline__ void load_batch(const T* __restrict__ D, int64_t ldd, int i0, int i_hi, int jb,
                                           int nvalid, T (&d)[StreamCfg<T, K, REBUILD>::NB][STREAM_CPL]) {
    constexpr int NB = StreamCfg<T, K, REBUILD>::NB;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int i = i0 + STREAM_WAVES * b;
        if (!CHECK || i < i_hi) {
            load4<(K <= D_LOADS_NT_KMAX && sizeof(T) == 4)>(D + (size_t)i * ldd + jb, FULL ? STREAM_CPL : nvalid, d[b]);
        } else {
#pragma unroll
            for (int s = 0; s < STREAM_CPL; ++s) d[b][s] = T(0);
        }
    }
}

// Threshold, residual and both product contributions of one loaded batch.
template <typename T, int K, bool REBUILD, bool CHECK>
__device__ __forceinline__ void compute_batch(
    const T (&d)[StreamCfg<T, K, REBUILD>::NB][STREAM_CPL], const T* __restrict__ AL, const T* __restrict__ Uf,
    int i0, int i_hi, T zeta, const T (&bl)[STREAM_CPL][K], const T (&vt)[STREAM_CPL][K],
    T (&y2)[STREAM_CPL][K], double& res, T& amax, typename AccOf<T>::type* __restrict__ P1t, int lane) {
    using Acc = typename AccOf<T>::type;
    constexpr int NB = StreamCfg<T, K, REBUILD>::NB;
    T p[NB * K];
    T rs = T(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int i = i0 + STREAM_WAVES * b;
#pragma unroll
        for (int t = 0; t < K; ++t) p[b * K + t] = T(0);
        if (!CHECK || i < i_hi) {
            T al[K], ut[K];
#pragma unroll
            for (int t = 0; t < K; ++t) {
                al[t] = REBUILD ? AL[(size_t)i * K + t] : T(0);
                ut[t] = Uf[(size_t)i * K + t];
            }
#pragma unroll
            for (int s = 0; s < STREAM_CPL; ++s) {
                const T dv = d[b][s];
                T x = dv;
                if constexpr (REBUILD) {
#pragma unroll
                    for (int t = 0; t < K; ++t) x = fma(-al[t], bl[s][t], x);
                }
                if constexpr (!REBUILD) amax = fmax(amax, fabs(x));   // L = 0: x = D_ij
                const bool big = fabs(x) > zeta;   // S_ij = x  (T_zeta keeps |x| > zeta)
                const T e = big ? T(0) : x;        // entry of E = D - L - S
                rs = fma(e, e, rs);
#pragma unroll
                for (int t = 0; t < K; ++t) {
                    y2[s][t] = fma(e, ut[t], y2[s][t]);
                    p[b * K + t] = fma(e, vt[s][t], p[b * K + t]);
                }
            }
        }
    }
    res += static_cast<double>(rs);
    const T tot = reduce_scatter64<NB * K>(p, lane);
    const int q = bitrev6(lane);
    if (q < NB * K) {
        const int b = q / K, t = q - (q / K) * K;
        const int i = i0 + STREAM_WAVES * b;
        if (i < i_hi) P1t[(size_t)i * K + t] = static_cast<Acc>(tot);
    }
}

// All rows of the tile for one wave. Full batches are software-pipelined: the
// loads of batch j+1 are issued before batch j is computed. FULL: the tile's
// 256 columns are all inside the matrix.
template <typename T, int K, bool REBUILD, bool FULL>
__device__ __forceinline__ void stream_rows(
    const T* __restrict__ D, int64_t ldd, const T* __restrict__ AL, const T* __restrict__ Uf,
    int i_first, int i_hi, int jb, int nvalid, T zeta, const T (&bl)[STREAM_CPL][K],
    const T (&vt)[STREAM_CPL][K], T (&y2)[STREAM_CPL][K], double& res, T& amax,
    typename AccOf<T>::type* __restrict__ P1t, int lane) {
    constexpr int NB = StreamCfg<T, K, REBUILD>::NB;
    constexpr int STEP = STREAM_WAVES * NB;
    int i0 = i_first;
    if (i0 + STREAM_WAVES * (NB - 1) < i_hi) {
        T cur[NB][STREAM_CPL], nxt[NB][STREAM_CPL];
        load_batch<T, K, REBUILD, FULL, false>(D, ldd, i0, i_hi, jb, nvalid, nxt);
        for (;;) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int s = 0; s < STREAM_CPL; ++s) cur[b][s] = nxt[b][s];
            const int i1 = i0 + STEP;
            const bool more = i1 + STREAM_WAVES * (NB - 1) < i_hi;
            if (more) load_batch<T, K, REBUILD, FULL, false>(D, ldd, i1, i_hi, jb, nvalid, nxt);
            compute_batch<T, K, REBUILD, false>(cur, AL, Uf, i0, i_hi, zeta, bl, vt, y2, res, amax, P1t, lane);
            i0 = i1;
            if (!more) break;
        }
    }
    for (; i0 < i_hi; i0 += STEP) {
        T cur[NB][STREAM_CPL];
        load_batch<T, K, REBUILD, FULL, true>(D, ldd, i0, i_hi, jb, nvalid, cur);
        compute_batch<T, K, REBUILD, true>(cur, AL, Uf, i0, i_hi, zeta, bl, vt, y2, res, amax, P1t, lane);
    }
}

// Waves per SIMD of the FP32 passes that miss three by a little: the
// initialisation's at K = 15 and the loop's at K = 10 (169 VGPRs of 168). The
// former, by the closing sums of an update, in whose Cholesky it spills 10 VGPRs
// for it: 10^4 x 10^4 171 -> 153 us a pass, 2 10^4 x 2 10^4 645 -> 540. The latter:
// 2 10^4 x 2 10^4, r = 10, plain schedule 14.31 -> 11.72 ms, 10^4 x 10^4 4.52 -> 4.02.
template <typename T, int K, bool REBUILD> constexpr int stream_min_waves() {
    return sizeof(T) == 4 && K == (REBUILD ? 10 : 15) ? 3 : 1;
}

template <typename T, int K, bool REBUILD>
__global__ __launch_bounds__(STREAM_THREADS, (stream_min_waves<T, K, REBUILD>())) void k_stream(
    const T* __restrict__ D, const T* __restrict__ AL, const T* __restrict__ BL, const T* __restrict__ Uf,
    const T* __restrict__ Vf, typename AccOf<T>::type* __restrict__ P1, typename AccOf<T>::type* __restrict__ P2,
    double* __restrict__ resid, Ctrl* __restrict__ ctrl, StreamGeom g) {
    using Acc = typename AccOf<T>::type;
    {   // instance blockIdx.y of a batched launch (slab 0: a single instance)
        const int64_t off = (int64_t)blockIdx.y * g.slab;
        D = moved(D, off);
        AL = moved(AL, off);
        BL = moved(BL, off);
        Uf = moved(Uf, off);
        Vf = moved(Vf, off);
        P1 = moved(P1, off);
        P2 = moved(P2, off);
        resid = moved(resid, off);
        ctrl = moved(ctrl, off);
    }
    if (!body_runs(ctrl, g.body)) return;
    const T zeta = static_cast<T>(ctrl->zeta);

    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int ct = tile % g.n_ct;
    const int rt = tile / g.n_ct;
    const int jb = ct * STREAM_TN + lane * STREAM_CPL;
    const int nvalid = min(max(g.n - jb, 0), STREAM_CPL);

    T bl[STREAM_CPL][K], vt[STREAM_CPL][K], y2[STREAM_CPL][K];
    if constexpr (REBUILD) load_panel_rows<T, STREAM_CPL, K>(BL, jb, nvalid, bl);
    load_panel_rows<T, STREAM_CPL, K>(Vf, jb, nvalid, vt);
#pragma unroll
    for (int s = 0; s < STREAM_CPL; ++s)
#pragma unroll
        for (int t = 0; t < K; ++t) {
            if constexpr (!REBUILD) bl[s][t] = T(0);
            y2[s][t] = T(0);
        }

    const int i_lo = rt * g.TM;
    const int i_hi = min(g.m, i_lo + g.TM);
    double res = 0.0;
    T amax = T(0);
    Acc* P1t = P1 + (size_t)ct * g.m * K;
    const bool full = (ct + 1) * STREAM_TN <= g.n;   // uniform per workgroup
    if (full)
        stream_rows<T, K, REBUILD, true>(D, g.ldd, AL, Uf, i_lo + wave, i_hi, jb, nvalid, zeta, bl, vt, y2, res,
                                         amax, P1t, lane);
    else
        stream_rows<T, K, REBUILD, false>(D, g.ldd, AL, Uf, i_lo + wave, i_hi, jb, nvalid, zeta, bl, vt, y2, res,
                                          amax, P1t, lane);

    // E^T Uf partial: sum the four waves' column partials through LDS.
    // the column partials; afterwards, scratch of pass_finishes_update
    constexpr int SM_BYTES = STREAM_TN * K * (int)sizeof(Acc);
    constexpr int FIN_BYTES = FINISH_LDS<K, STREAM_THREADS>() * (int)sizeof(double);
    __shared__ __align__(16) unsigned char sm_raw[SM_BYTES > FIN_BYTES ? SM_BYTES : FIN_BYTES];
    Acc* sm = reinterpret_cast<Acc*>(sm_raw);
    __shared__ double red[STREAM_WAVES];
    for (int w = 0; w < STREAM_WAVES; ++w) {
        if (wave == w) {
#pragma unroll
            for (int s = 0; s < STREAM_CPL; ++s)
#pragma unroll
                for (int t = 0; t < K; ++t) {
                    const int idx = (lane * STREAM_CPL + s) * K + t;
                    sm[idx] = (w == 0) ? static_cast<Acc>(y2[s][t]) : sm[idx] + static_cast<Acc>(y2[s][t]);
                }
        }
        __syncthreads();
    }
    for (int idx = threadIdx.x; idx < STREAM_TN * K; idx += STREAM_THREADS) {
        const int col = ct * STREAM_TN + idx / K;
        if (col < g.n) P2[((size_t)rt * g.n + col) * K + (idx % K)] = sm[idx];
    }
    const double rtot = block_sum_256(res, red);
    if (threadIdx.x == 0) resid[tile] = rtot;
    if constexpr (!REBUILD) {
        // max |D_ij| over the tile, behind the residuals of all tiles
        double v = static_cast<double>(amax);
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, WAVE));
        if (lane == 0) red[wave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double mx = red[0];
            for (int w = 1; w < STREAM_WAVES; ++w) mx = fmax(mx, red[w]);
            resid[gridDim.x + tile] = mx;
        }
    }
    pass_finishes_update<K, STREAM_THREADS>(ctrl, g, (int64_t)blockIdx.y * g.slab, reinterpret_cast<double*>(sm_raw));
}

// Dense L = AL BL^T and S = T_zeta(D - L) (outputs of Algorithm 1).
//
// Bound by memory: D read (only for S), L and S written. A wave covers
// 64 x VW columns with one 16-byte access per lane and row and keeps its rows
// of BL in registers; the row of AL is wave-uniform (scalar loads). The four
// waves of a workgroup take interleaved rows, MAT_U of them in flight. The
// accesses ask only for element alignment (the hardware takes 16-byte
// accesses at any 4-byte address), so odd strides run the same code; lanes
// past the last whole vector of a row go element by element.
//
// WHOLE: every row of the outputs starts at a multiple of MAT_SECTOR bytes, so
// that a wave's 1 KB of a row is whole memory sectors: the outputs, which no
// kernel reads back, are stored non-temporally. Otherwise neighbouring column
// tiles share a sector at their edges: they go to the same XCD (xcd_tile) at about
// the same time, through its L2, which puts the two halves together; beyond
// MAT_FINE_KMAX columns half as many workgroups then are faster (what each loads
// first, its rows of BL, is not whole sectors either).
//
// L and S, a call: m = n = 10^4, r = 5, FP32 (1.2 GB): 421 -> 251 us (the kernel
// 4.9 TB/s; a plain copy reaches 5.2), FP64 640 -> 469. FP64, 10^4 x 3011, r = 1
// (rows at any multiple of 8 bytes): 178 -> 173 us; 12000 x 2436, r = 9: 292 -> 182
// (with twice the workgroups 188). 4096 workgroups took 254, 487, 179 and 182; the
// ragged ones stored non-temporally, in plain order, 196 and 185.
// L alone, 10^4 x 10^4, FP32: 240 -> 81 us, where D is not read at all.
constexpr int MAT_U = 4;                           // rows in flight per wave
constexpr int MAT_ROWS = MAT_U * STREAM_WAVES;     // rows of a workgroup per step
constexpr int MAT_TILES = 8192;                    // workgroups aimed at (32 per CU)
constexpr int MAT_SECTOR = 64;
constexpr int MAT_FINE_KMAX = 6;

// (The vector type is named, not deduced: deduction drops its element alignment.)
template <bool NT, typename T>
__device__ __forceinline__ void mat_store(typename Vec16u<T>::type v, typename Vec16u<T>::type* p) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// MAT_U rows i0, i0 + 4, ... of one wave; CHECK: some may lie at or past i_hi.
template <typename T, int K, bool SOUT, bool WHOLE, bool CHECK>
__device__ __forceinline__ void materialize_rows(const T* __restrict__ D, int64_t ldd, const T* __restrict__ AL,
                                                 T* __restrict__ Lo, int64_t ldl, T* __restrict__ So, int64_t lds,
                                                 int i0, int i_hi, int j, int nv, T zeta,
                                                 const T (&b)[16 / sizeof(T)][K]) {
    constexpr int VW = 16 / (int)sizeof(T);
    typedef typename Vec16u<T>::type VecT;
    VecT d[MAT_U];
    if constexpr (SOUT) {
#pragma unroll
        for (int u = 0; u < MAT_U; ++u) {
            const int i = i0 + u * STREAM_WAVES;
            if (CHECK && i >= i_hi) continue;
            const T* p = D + (size_t)i * ldd + j;
            if (nv == VW) {
                d[u] = *reinterpret_cast<const VecT*>(p);
            } else {
#pragma unroll
                for (int s = 0; s < VW; ++s) d[u][s] = s < nv ? p[s] : T(0);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < MAT_U; ++u) {
        const int i = i0 + u * STREAM_WAVES;
        if (CHECK && i >= i_hi) continue;
        VecT l, o;
#pragma unroll
        for (int s = 0; s < VW; ++s) {
            T v = T(0);
#pragma unroll
            for (int t = 0; t < K; ++t) v = fma(AL[(size_t)i * K + t], b[s][t], v);
            l[s] = v;
            if constexpr (SOUT) {
                const T x = d[u][s] - v;
                o[s] = fabs(x) > zeta ? x : T(0);
            }
        }
        if (Lo) {
            T* p = Lo + (size_t)i * ldl + j;
            if (nv == VW) {
                mat_store<WHOLE, T>(l, reinterpret_cast<VecT*>(p));
            } else {
#pragma unroll
                for (int s = 0; s < VW; ++s)
                    if (s < nv) p[s] = l[s];
            }
        }
        if constexpr (SOUT) {
            T* p = So + (size_t)i * lds + j;
            if (nv == VW) {
                mat_store<WHOLE, T>(o, reinterpret_cast<VecT*>(p));
            } else {
#pragma unroll
                for (int s = 0; s < VW; ++s)
                    if (s < nv) p[s] = o[s];
            }
        }
    }
}

template <typename T, int K, bool SOUT, bool WHOLE>
__global__ __launch_bounds__(STREAM_THREADS) void k_materialize(
    const T* __restrict__ D, const T* __restrict__ AL, const T* __restrict__ BL, T zeta, T* __restrict__ Lo,
    T* __restrict__ So, int64_t ldd, int64_t ldl, int64_t lds, int m, int n, int n_ct, int TM) {
    constexpr int VW = 16 / (int)sizeof(T);
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int tile = WHOLE ? blockIdx.x : xcd_tile(blockIdx.x, gridDim.x);
    const int ct = tile % n_ct, rt = tile / n_ct;
    const int j = (ct * WAVE + lane) * VW;
    const int nv = min(max(n - j, 0), VW);
    if (nv == 0) return;
    T b[VW][K];
    load_panel_rows<T, VW, K>(BL, j, nv, b);
    const int i_hi = min(m, (rt + 1) * TM);
    int i0 = rt * TM + wave;
    for (; i0 + STREAM_WAVES * (MAT_U - 1) < i_hi; i0 += MAT_ROWS)
        materialize_rows<T, K, SOUT, WHOLE, false>(D, ldd, AL, Lo, ldl, So, lds, i0, i_hi, j, nv, zeta, b);
    if (i0 < i_hi) materialize_rows<T, K, SOUT, WHOLE, true>(D, ldd, AL, Lo, ldl, So, lds, i0, i_hi, j, nv, zeta, b);
}

// Read-bandwidth reference: every 16-byte word of [p, p + n16) read once,
// eight loads in flight per thread, no arithmetic beyond a sum that is
// written only if it equals an impossible value (so the loads stay).
__global__ __launch_bounds__(256) void k_read_probe(const float4* __restrict__ p, int64_t n16, float* sink) {
    constexpr int U = 8;
    float acc = 0.f;
    const int64_t stride = (int64_t)gridDim.x * 256 * U;
    for (int64_t i = (int64_t)blockIdx.x * 256 * U + threadIdx.x; i < n16; i += stride) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = i + (int64_t)u * 256;
            v[u] = j < n16 ? p[j] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc += (v[u].x + v[u].y) + (v[u].z + v[u].w);
    }
    if (acc == -1.2345e-38f) sink[blockIdx.x] = acc;
}

template <typename T, bool REBUILD>
hipError_t stream_dispatch(const StreamArgs& a, int K, hipStream_t s) {
    using Acc = typename AccOf<T>::type;
    const dim3 grid((unsigned)(a.n_ct * a.n_rt), a.batch > 1 ? (unsigned)a.batch : 1u), block(STREAM_THREADS);
    StreamGeom geom;
    geom.slab = a.batch > 1 ? a.slab : 0;
    geom.ldd = a.ldd;
    geom.m = a.m;
    geom.n = a.n;
    geom.TM = a.TM;
    geom.n_ct = a.n_ct;
    geom.n_rt = a.n_rt;
    geom.body = a.body;
    geom.post_gpart = a.post_gpart;
    geom.post_small = a.post_small;
    geom.post_gU = a.post_gU;
    geom.post_gV = a.post_gV;
    switch (K) {
#define RPCA_CASE(KK)                                                                                      \
    case KK:                                                                                               \
        hipLaunchKernelGGL((k_stream<T, KK, REBUILD>), grid, block, 0, s, static_cast<const T*>(a.D),      \
                           static_cast<const T*>(a.AL), static_cast<const T*>(a.BL),                       \
                           static_cast<const T*>(a.Uf), static_cast<const T*>(a.Vf), static_cast<Acc*>(a.P1), \
                           static_cast<Acc*>(a.P2), a.resid, a.ctrl, geom);                                \
        break;
        RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5) RPCA_CASE(6)
        RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10) RPCA_CASE(11) RPCA_CASE(12)
        RPCA_CASE(13) RPCA_CASE(14) RPCA_CASE(15) RPCA_CASE(16)
#undef RPCA_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, bool SOUT, bool WHOLE>
hipError_t materialize_tiles(const MaterializeArgs& a, int K, hipStream_t s) {
    constexpr int TN = WAVE * (16 / (int)sizeof(T));
    const int n_ct = (a.n + TN - 1) / TN;
    const int most = (a.m + MAT_ROWS - 1) / MAT_ROWS;
    int n_rt = (WHOLE || K <= MAT_FINE_KMAX ? MAT_TILES : MAT_TILES / 2) / n_ct;
    n_rt = n_rt < 1 ? 1 : (n_rt < most ? n_rt : most);
    int TM = (a.m + n_rt - 1) / n_rt;
    TM = (TM + MAT_ROWS - 1) / MAT_ROWS * MAT_ROWS;
    n_rt = (a.m + TM - 1) / TM;
    const dim3 grid((unsigned)((int64_t)n_ct * n_rt)), block(STREAM_THREADS);
    switch (K) {
#define RPCA_CASE(KK) \
    case KK:                                                                                                   \
        hipLaunchKernelGGL((k_materialize<T, KK, SOUT, WHOLE>), grid, block, 0, s, static_cast<const T*>(a.D), \
                           static_cast<const T*>(a.AL), static_cast<const T*>(a.BL), static_cast<T>(a.zeta),  \
                           static_cast<T*>(a.L_out), static_cast<T*>(a.S_out), a.ldd, a.ldl, a.lds, a.m, a.n, \
                           n_ct, TM);                                                                         \
        break;
        RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5) RPCA_CASE(6)
        RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10) RPCA_CASE(11) RPCA_CASE(12)
        RPCA_CASE(13) RPCA_CASE(14) RPCA_CASE(15) RPCA_CASE(16)
#undef RPCA_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, bool SOUT> hipError_t materialize_dispatch(const MaterializeArgs& a, int K, hipStream_t s) {
    const auto whole = [](const void* p, int64_t ld) {
        return !p || ((uintptr_t)p % MAT_SECTOR == 0 && (ld * (int64_t)sizeof(T)) % MAT_SECTOR == 0);
    };
    return whole(a.L_out, a.ldl) && whole(a.S_out, a.lds) ? materialize_tiles<T, SOUT, true>(a, K, s)
                                                          : materialize_tiles<T, SOUT, false>(a, K, s);
}

template <typename T, bool REBUILD>
int stream_occupancy_t(int K) {
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (K) {
#define RPCA_CASE(KK)                                                                                   \
    case KK:                                                                                            \
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_stream<T, KK, REBUILD>, STREAM_THREADS, 0); \
        break;
        RPCA_CASE(1) RPCA_CASE(2) RPCA_CASE(3) RPCA_CASE(4) RPCA_CASE(5) RPCA_CASE(6)
        RPCA_CASE(7) RPCA_CASE(8) RPCA_CASE(9) RPCA_CASE(10) RPCA_CASE(11) RPCA_CASE(12)
        RPCA_CASE(13) RPCA_CASE(14) RPCA_CASE(15) RPCA_CASE(16)
#undef RPCA_CASE
        default: break;
    }
    return (e == hipSuccess && n > 0) ? n : 1;
}

}  // namespace

int stream_occupancy(int K, int dtype, bool rebuild) {
    if (dtype == 1) return rebuild ? stream_occupancy_t<float, true>(K) : stream_occupancy_t<float, false>(K);
    return rebuild ? stream_occupancy_t<double, true>(K) : stream_occupancy_t<double, false>(K);
}

hipError_t launch_stream(const StreamArgs& a, int K, int dtype, bool rebuild, hipStream_t s) {
    if (dtype == 1) return rebuild ? stream_dispatch<float, true>(a, K, s) : stream_dispatch<float, false>(a, K, s);
    return rebuild ? stream_dispatch<double, true>(a, K, s) : stream_dispatch<double, false>(a, K, s);
}

hipError_t launch_read_probe(const void* data, int64_t bytes, float* sink, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_read_probe, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const float4*>(data),
                       bytes / 16, sink);
    return hipGetLastError();
}

hipError_t launch_materialize(const MaterializeArgs& a, int K, int dtype, hipStream_t s) {
    if (dtype == 1) return a.S_out ? materialize_dispatch<float, true>(a, K, s) : materialize_dispatch<float, false>(a, K, s);
    return a.S_out ? materialize_dispatch<double, true>(a, K, s) : materialize_dispatch<double, false>(a, K, s);
}

}  // namespace rpca
