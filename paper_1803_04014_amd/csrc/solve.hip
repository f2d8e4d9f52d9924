// solve.hip -- a consumer of the GEMM: mixed-precision iterative refinement
// for A X = B (the technique the paper puts its precision refinement next
// to, Sec. V), with the O(n^3) work of the factorisation on the matrix
// cores through mfg_gemm.
//
//   LU:  right-looking blocked LU with partial pivoting of an FP32 copy of
//        A, panels of kNb = 64 columns, a panel in sub-panels of 8 to 32
//        columns, each factored by one workgroup in registers (column by
//        column: pivot search, row exchange, scaling by the pivot's
//        reciprocal as in LAPACK's unblocked LU, rank-1 update); the panel's
//        row exchanges are applied to the rest of the matrix in the launch
//        that solves the block row with the panel's unit lower triangle
//        (U12 = L11^-1 A12), and the trailing matrix is updated
//        A22 -= L21 U12 by one mfg_gemm call in the caller's mode (F32, F16,
//        or a refined split: the precision of the factorisation).
//   solve with the factors: the row permutation (one gather), then forward
//        and backward substitution by blocks of kNb rows, one launch each:
//        a wavefront per block and right-hand side, waiting for the unknowns
//        of the blocks before it.
//   refinement: x0 from the factors; then r = b - A x in FP64, the normwise
//        backward error max_j |r_j|_inf / (|A|_inf |x_j|_inf + |b_j|_inf),
//        and while it is above the tolerance a correction d solved in FP32
//        from r and x += d in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>
#include <vector>

#include "internal.h"
#include "runtime.h"

namespace mfg {

namespace {

constexpr int kNb = 64;
constexpr int kPanelThreads = 1024;

// One panel A[j:n, j:j+w] (w <= kNb), factored in place with partial pivoting.
// ipiv[j + c] receives the row swapped with row j + c (0-based); info (if no
// earlier column had one) the 1-based index of the first exactly-zero pivot.
__global__ __launch_bounds__(kPanelThreads) void lu_panel(int64_t n, float* A, int64_t lda, int64_t j, int w,
                                                         int32_t* ipiv, int32_t* info) {
    __shared__ float prow[kNb];
    __shared__ float wv[kPanelThreads / 64];
    __shared__ int64_t wi[kPanelThreads / 64];
    __shared__ int64_t piv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int c = 0; c < w; ++c) {
        const int64_t col = j + c;
        // pivot: the largest |A[r, col]| over r >= col, the first such row on ties
        float best = -1.0f;
        int64_t bi = n;
        for (int64_t r = col + tid; r < n; r += kPanelThreads) {
            const float v = fabsf(A[r * lda + col]);
            if (v > best) best = v, bi = r;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const float ov = __shfl_xor(best, off);
            const int64_t oi = __shfl_xor(bi, off);
            if (ov > best || (ov == best && oi < bi)) best = ov, bi = oi;
        }
        if (lane == 0) wv[wave] = best, wi[wave] = bi;
        __syncthreads();
        if (tid == 0) {
            float b = wv[0];
            int64_t i = wi[0];
            for (int q = 1; q < kPanelThreads / 64; ++q)
                if (wv[q] > b || (wv[q] == b && wi[q] < i)) b = wv[q], i = wi[q];
            if (i >= n) i = col;  // (a column of NaNs only: keep the diagonal)
            piv = i;
            ipiv[col] = (int32_t)i;
            if (A[i * lda + col] == 0.0f && *info == 0) *info = (int32_t)(col + 1);
        }
        __syncthreads();
        const int64_t p = piv;
        if (p != col && tid < w) {
            const float t = A[col * lda + j + tid];
            A[col * lda + j + tid] = A[p * lda + j + tid];
            A[p * lda + j + tid] = t;
        }
        __syncthreads();
        if (tid < w) prow[tid] = A[col * lda + j + tid];
        __syncthreads();
        const float pv = prow[c];
        if (pv != 0.0f) {
            const float rp = 1.0f / pv;  // the column is scaled by the pivot's reciprocal
            for (int64_t r = col + 1 + tid; r < n; r += kPanelThreads) {
                float* row = A + r * lda + j;
                const float l = row[c] * rp;
                row[c] = l;
                for (int cc = c + 1; cc < w; ++cc) row[cc] = __builtin_fmaf(-l, prow[cc], row[cc]);
            }
        }
        __syncthreads();
    }
}

// The rows a panel of kNb columns exchanges, as moves (row indices from the
// panel's first row): after the panel is factored, row t < w of every other
// column holds what row top[t] held before it, and row dst[i] (below the
// panel's w rows, i < ndisp <= w) what row src[i] held.  Applied as one gather
// and one scatter, a column's rows are all loaded before any is stored.
struct LuMoves {
    int32_t ndisp;
    int32_t top[kNb], dst[kNb], src[kNb];
};

// One sub-panel A[jj : jj + rows, jj : jj + w] (w <= W) of the panel whose
// columns are [j, j + cw): factored with partial pivoting in the registers of
// one workgroup, its row exchanges applied to the panel's other columns, and
// the block row right of it solved with its unit lower triangle
// (U12 = L11^-1 A12).
//
// Bound by latency: one column's pivot search decides the next column.  The
// threads' registers hold up to 64 K elements: 512 threads with 128 each
// (2048 rows x 32, 4096 x 16), 256 (a wavefront per SIMD) for up to 1024 rows x
// 32, so a panel of 64 columns is 2 or 4 sub-panels by its height.
// At 2048 rows 54 us per 32 columns (four sub-panels of 8 with launches of
// their own for the exchanges took 94 us and 11 gaps between launches): about
// 10 us for the rows to arrive (256 KB at what one CU can have outstanding),
// 0.8 us per column, 3 us per group's update, 10 us for the exchanges, the
// solve and the stores.  4096 x 16: 38 us (two of 8: 47).
//
// Thread t holds rows i = t + NT q (row jj + i), x[q][0 .. W-1].  Rows are
// never exchanged in registers: pos[q] is the row's place after the exchanges
// so far (-1: past the matrix), and a row goes to its place when it is stored.
// The columns go in groups of 8 (at positions 0 .. 7; after each group the
// array rotates by 8).  Per column:
//   - each wavefront finds its largest |value| at or below the diagonal, the
//     first place on ties (fmaxf ignores NaN); the lane holding it writes the
//     row's entries of the group to the wavefront's LDS slot;
//   - one barrier; every thread reduces the candidates by the same rule,
//     places are exchanged, and every row below the diagonal is scaled by the
//     pivot's reciprocal and its entries of the group updated.
// After a group its 8 pivot rows go to LDS, each wavefront solves the columns
// to come with the group's unit lower triangle (lane = column), and every row
// takes the 8 multiply-adds per column, the solved entries by readlane.  (Eight
// columns at a time rather than all at once: a quarter of the LDS reads per
// column, and nothing but the group's entries between two searches.)
// The LDS slots alternate by column parity: a slot is written again two
// columns later, by threads that passed the barrier of the column in between,
// which every thread reaches only after reading it.  The same operations in
// the same order per element as lu_panel.
//
// org (n ints, rows from j): where each row of the panel came from, carried
// from sub-panel to sub-panel; the last one writes the panel's moves.
template <int CTRL>
__device__ __forceinline__ int dpp_max_i32(int v) {
    const int o = __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
    return max(o, v);
}
template <int CTRL>
__device__ __forceinline__ int dpp_min_i32(int v) {
    const int o = __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
    return min(o, v);
}
// Over the wavefront: inside each 16-lane row by quad_perm xor 1, xor 2, then
// row_ror 4, row_ror 8; the four rows by readlane.
__device__ __forceinline__ int wave_max_i32(int v) {
    v = dpp_max_i32<0x128>(dpp_max_i32<0x124>(dpp_max_i32<0x4E>(dpp_max_i32<0xB1>(v))));
    const int a = max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
    return max(a, max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ int wave_min_i32(int v) {
    v = dpp_min_i32<0x128>(dpp_min_i32<0x124>(dpp_min_i32<0x4E>(dpp_min_i32<0xB1>(v))));
    const int a = min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
    return min(a, min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

__device__ __forceinline__ float lane_of(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// All of this thread's loads and stores done, then the workgroup's barrier.
__device__ __forceinline__ void memory_barrier() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Over N = 4 or 8 values held by lanes 0 .. N-1 and repeated by the lanes after
// them: by quad_perm xor 1, xor 2, then row_half_mirror.
template <int N>
__device__ __forceinline__ int keys_max_i32(int v) {
    v = dpp_max_i32<0x4E>(dpp_max_i32<0xB1>(v));
    if constexpr (N > 4) v = dpp_max_i32<0x141>(v);
    return __builtin_amdgcn_readfirstlane(v);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

// This wavefront's LDS writes before its reads by other lanes, and the reverse.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int W, int Q, int NT>
__global__ __launch_bounds__(NT, 1) void lu_sub(int rows, const float* in, int64_t ldin, float* A, int64_t lda,
                                              int64_t j, int64_t jj, int w,
                                              int cw, int vec, int32_t* ipiv, int32_t* info, int32_t* org,
                                              LuMoves* moves) {
    static_assert(W % 8 == 0 && W <= kNb, "groups of eight columns");
    constexpr int NW = NT / 64, G = 8, NG = W / G;
    static_assert(NW == 4 || NW == 8, "the wavefronts' candidate rows fit one register");
    __shared__ __attribute__((aligned(16))) int2 skey[2][NW];             // |value| bits (-1: none), place
    __shared__ __attribute__((aligned(16))) float srow[2][NW + 1][G];     // candidates, then the diagonal row
    __shared__ __attribute__((aligned(16))) float spiv[2][G][W];          // a group's pivot rows
    __shared__ int mtop[W], mdst[W], msrc[W], mcount, pcount;
    __shared__ __attribute__((aligned(16))) float L[W][W];
    __shared__ float T[W][kNb];
    // a wavefront's rows on their way between memory (W / 4 lanes per row, whole
    // lines) and registers (a lane per row)
    constexpr int kRowLanes = W / 4, kRowsAt = 64 / kRowLanes, kStage = W + 4;
    __shared__ __attribute__((aligned(16))) float stage[NW][64][kStage];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rl = lane / kRowLanes, cl = lane % kRowLanes * 4;
    const bool whole = vec && w == W;  // (in, a copy, is aligned where A is)
    const int left = (int)(jj - j);  // columns of the panel before the sub-panel
    float x[Q][W];
    int pos[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = tid + NT * q;
        pos[q] = i < rows ? i : -1;
        if (!whole) {
            const float* rp = in + (i < rows ? i : 0) * ldin;
#pragma unroll
            for (int k = 0; k < W; ++k) x[q][k] = k < w ? rp[k] : 0.0f;
        }
    }
    if (whole) {
        floatx4 piece[Q][kRowLanes];  // (the vector type: an array of float4 stays in memory)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int e = 0; e < kRowLanes; ++e) {
                const int i = NT * q + wave * 64 + kRowsAt * e + rl;
                piece[q][e] = *reinterpret_cast<const floatx4*>(in + min(i, rows - 1) * ldin + cl);
            }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            wave_sync();
#pragma unroll
            for (int e = 0; e < kRowLanes; ++e)
                *reinterpret_cast<floatx4*>(&stage[wave][kRowsAt * e + rl][cl]) = piece[q][e];
            wave_sync();
#pragma unroll
            for (int k = 0; k < W; k += 4) {
                const float4 v = *reinterpret_cast<const float4*>(&stage[wave][lane][k]);
                x[q][k] = v.x, x[q][k + 1] = v.y, x[q][k + 2] = v.z, x[q][k + 3] = v.w;
            }
        }
    }
    if (tid == 0) mcount = 0, pcount = 0;
    int first0 = 0;  // (thread 0) 1 + the first column with a zero pivot

#pragma unroll 1
    for (int g = 0; g < NG; ++g) {
        uint32_t used = 0;  // the group's columns that updated the rows below
        auto column = [&](auto ccst) {
            constexpr int cc = decltype(ccst)::value, buf = cc & 1;
            const int c = G * g + cc;
            if (c >= w) return;
            float m = -1.0f;
#pragma unroll
            for (int q = 0; q < Q; ++q) m = fmaxf(m, pos[q] >= c ? fabsf(x[q][cc]) : -1.0f);
            int mp = INT32_MAX;
#pragma unroll
            for (int q = 0; q < Q; ++q) mp = min(mp, pos[q] >= c && fabsf(x[q][cc]) == m ? pos[q] : INT32_MAX);
            asm("" : "+v"(mp));  // (ready before the reduction, not after it)
            const int bits = m >= 0.0f ? __builtin_bit_cast(int, m) : -1;
            const int wm = wave_max_i32(bits);
            const uint64_t at = __ballot(bits == wm);
            int wi = -2;  // no place
            if (wm >= 0) {
                if ((at & (at - 1)) == 0) wi = __builtin_amdgcn_readlane(mp, __builtin_ctzll(at));
                else wi = wave_min_i32(bits == wm ? mp : INT32_MAX);
            }
            if (lane == 0) skey[buf][wave] = make_int2(wm, wi);
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (pos[q] == wi) {
#pragma unroll
                    for (int k = 0; k < G; k += 4)
                        *reinterpret_cast<float4*>(&srow[buf][wave][k]) =
                            make_float4(x[q][k], x[q][k + 1], x[q][k + 2], x[q][k + 3]);
                }
            __syncthreads();
            // every wavefront's key and row with one LDS read each: lane q (and
            // q + NW, ...) holds key q, lane 8 q + k entry k of row q
            const int2 key = skey[buf][lane % NW];
            const float cand = (&srow[buf][0][0])[lane % (NW * G)];
            const int pm = keys_max_i32<NW>(key.x);
            const float ra = 1.0f / __builtin_bit_cast(float, pm);
            int pi = c;
            float pr[G];
            if (pm >= 0) {
                uint64_t best = __ballot(key.x == pm) & ((1ull << NW) - 1);
                if ((best & (best - 1)) != 0) {
                    const int first = wave_min_i32(key.x == pm ? key.y : INT32_MAX);
                    best = __ballot(key.x == pm && key.y == first) & ((1ull << NW) - 1);
                }
                const int pw = __builtin_ctzll(best);
                pi = __builtin_amdgcn_readlane(key.y, pw);
#pragma unroll
                for (int k = cc; k < G; ++k) pr[k] = lane_of(cand, pw * G + k);
            } else {  // no candidate (every |value| NaN): the diagonal row
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (pos[q] == c) {
#pragma unroll
                        for (int k = 0; k < G; ++k) srow[buf][NW][k] = x[q][k];
                    }
                __syncthreads();
#pragma unroll
                for (int k = cc; k < G; ++k) pr[k] = lane_of(srow[buf][NW][k], 0);
            }
            const float rp = pm < 0 ? pr[cc] : __builtin_copysignf(ra, pr[cc]);
            if (tid == 0) ipiv[jj + c] = (int32_t)(jj + pi);
#pragma unroll
            for (int q = 0; q < Q; ++q) pos[q] = pos[q] == pi ? c : pos[q] == c ? pi : pos[q];
            if (pm != 0) {  // the pivot is not zero
                used |= 1u << cc;
#pragma unroll
                for (int q = 0; q < Q; ++q) {  // (selects: a branch around them costs more, and copies)
                    const float l = x[q][cc] * rp;
                    const bool below = pos[q] > c;
                    x[q][cc] = below ? l : x[q][cc];
#pragma unroll
                    for (int k = cc + 1; k < G; ++k) {
                        const float v = __builtin_fmaf(-l, pr[k], x[q][k]);
                        x[q][k] = below ? v : x[q][k];
                    }
                }
            } else if (first0 == 0) {
                first0 = (int32_t)(jj + c + 1);
            }
        };
        [&]<int... Cs>(std::integer_sequence<int, Cs...>) {
            (column(std::integral_constant<int, Cs>{}), ...);
        }(std::make_integer_sequence<int, G>{});
        if constexpr (NG > 1) {
            const int c0 = G * g;
            if (c0 + G < w) {  // columns to come, at positions G ..
                // (alternating buffers: the one of two groups ago was read before 8 barriers)
                float(*sp)[W] = spiv[g & 1];
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (pos[q] >= c0 && pos[q] < c0 + G) {
#pragma unroll
                        for (int k = 0; k < W; k += 4)
                            *reinterpret_cast<float4*>(&sp[pos[q] - c0][k]) =
                                make_float4(x[q][k], x[q][k + 1], x[q][k + 2], x[q][k + 3]);
                    }
                __syncthreads();
                float u[G], l[G][G];
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    u[i] = sp[i][lane % W];
                    const float4 l0 = *reinterpret_cast<const float4*>(&sp[i][0]);
                    const float4 l1 = *reinterpret_cast<const float4*>(&sp[i][4]);
                    l[i][0] = l0.x, l[i][1] = l0.y, l[i][2] = l0.z, l[i][3] = l0.w;
                    l[i][4] = l1.x, l[i][5] = l1.y, l[i][6] = l1.z, l[i][7] = l1.w;
                }
#pragma unroll
                for (int k = 0; k < G - 1; ++k) {
                    const bool on = used >> k & 1;
#pragma unroll
                    for (int i = k + 1; i < G; ++i) {
                        const float t = __builtin_fmaf(-l[i][k], u[k], u[i]);
                        u[i] = on ? t : u[i];
                    }
                }
                // the pivot rows are the solved ones (by LDS to the lanes that hold
                // them), the rows below take the group's multiples
                wave_sync();
#pragma unroll
                for (int i = 0; i < G; ++i)
                    if (lane < W) stage[wave][i][lane] = u[i];
                wave_sync();
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (pos[q] >= c0 && pos[q] < c0 + G) {
#pragma unroll
                        for (int k = G; k < W; k += 4) {
                            if (k / G + g >= NG) continue;  // uniform
                            const float4 v = *reinterpret_cast<const float4*>(&stage[wave][pos[q] - c0][k]);
                            x[q][k] = v.x, x[q][k + 1] = v.y, x[q][k + 2] = v.z, x[q][k + 3] = v.w;
                        }
                    }
#pragma unroll
                for (int b = 1; b < NG; ++b) {
                    if (b + g >= NG) continue;  // uniform
                    float uk[G][G];
#pragma unroll
                    for (int k = 0; k < G; ++k)
#pragma unroll
                        for (int e = 0; e < G; ++e) uk[k][e] = lane_of(u[k], G * b + e);
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if (pos[q] >= c0 + G) {
#pragma unroll
                            for (int k = 0; k < G; ++k) {
                                if (!(used >> k & 1)) continue;  // uniform
#pragma unroll
                                for (int e = 0; e < G; ++e)
                                    x[q][G * b + e] = __builtin_fmaf(-x[q][k], uk[k][e], x[q][G * b + e]);
                            }
                        }
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                float t[G];
#pragma unroll
                for (int k = 0; k < G; ++k) t[k] = x[q][k];
#pragma unroll
                for (int k = 0; k < W - G; ++k) x[q][k] = x[q][k + G];
#pragma unroll
                for (int k = 0; k < G; ++k) x[q][W - G + k] = t[k];
            }
        }
    }
    if (tid == 0 && first0 != 0 && *info == 0) *info = first0;

    // the rows that moved, and L11
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = tid + NT * q;
        if (i >= rows) continue;
        if (pos[q] < w) {
            mtop[pos[q]] = i;
#pragma unroll
            for (int k = 0; k < W; k += 4)
                *reinterpret_cast<float4*>(&L[pos[q]][k]) = make_float4(x[q][k], x[q][k + 1], x[q][k + 2], x[q][k + 3]);
        } else if (pos[q] != i) {  // at most w such rows
            const int at = atomicAdd(&mcount, 1);
            mdst[at] = pos[q], msrc[at] = i;
        }
    }
    __syncthreads();
    if (cw > w) {
        // The panel's other columns (`left` before, the rest after the
        // sub-panel): rows top[] and src[] all loaded, then stored (right of the
        // sub-panel the top rows go to T for the solve).
        const int nm = w + mcount;
        constexpr int kPer = 2 * W * kNb / NT;
        float v[kPer];
        const int col = tid & (kNb - 1), r0 = tid / kNb;  // column of the panel, first row of this thread
        const bool mine = col < cw && (col < left || col >= left + w);
        float* cp = A + jj * lda + j + col;
        const float* lp = mine ? cp : A + jj * lda + jj;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int r = r0 + u * (NT / kNb);
            const int top = mtop[min(r, w - 1)], src = msrc[min(max(r - w, 0), W - 1)];
            v[u] = lp[(int64_t)(r >= nm ? 0 : r < w ? top : src) * lda];  // (no branch around a load)
        }
        memory_barrier();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int r = r0 + u * (NT / kNb);
            if (!mine || r >= nm) continue;
            if (r < w && col >= left) T[r][col] = v[u];
            else cp[(int64_t)(r < w ? r : mdst[r - w]) * lda] = v[u];
        }
        __syncthreads();
        if (tid >= left + w && tid < cw) {  // (then w == W)
            float y[W];
#pragma unroll
            for (int i = 0; i < W; ++i) y[i] = T[i][tid];
#pragma unroll
            for (int k4 = 0; k4 < W; k4 += 4)
#pragma unroll
                for (int i = k4 + 1; i < W; ++i) {
                    const float4 l4 = *reinterpret_cast<const float4*>(&L[i][k4]);
                    const float l[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                    for (int k = k4; k < k4 + 4 && k < i; ++k) y[i] = __builtin_fmaf(-l[k - k4], y[k], y[i]);
                }
#pragma unroll
            for (int i = 0; i < W; ++i) A[(jj + i) * lda + j + tid] = y[i];
        }
    }
    // this sub-panel's origins composed with those before it
    if (left + w == cw) {
        if (tid < left) moves->top[tid] = org[tid];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = tid + NT * q;
            if (i >= rows) continue;
            const int from = left == 0 ? i : org[left + i], at = left + pos[q];
            if (pos[q] < w) {
                moves->top[at] = from;
            } else if (from != at) {  // at most cw such rows
                const int e = atomicAdd(&pcount, 1);
                moves->dst[e] = at, moves->src[e] = from;
            }
        }
        __syncthreads();
        if (tid == 0) moves->ndisp = pcount;
    } else {
        int from[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = tid + NT * q;
            from[q] = left == 0 || i >= rows ? left + i : org[left + i];
        }
        if (left != 0) memory_barrier();
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (tid + NT * q < rows) org[left + pos[q]] = from[q];
    }
    // the factored rows to their places
    if (whole) {
        int* place = reinterpret_cast<int*>(&stage[wave][0][W]);  // (rows' padding)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            wave_sync();
#pragma unroll
            for (int k = 0; k < W; k += 4)
                *reinterpret_cast<float4*>(&stage[wave][lane][k]) =
                    make_float4(x[q][k], x[q][k + 1], x[q][k + 2], x[q][k + 3]);
            place[lane * kStage] = pos[q];
            wave_sync();
#pragma unroll
            for (int e = 0; e < kRowLanes; ++e) {
                const int r = kRowsAt * e + rl, at = place[r * kStage];
                const float4 v = *reinterpret_cast<const float4*>(&stage[wave][r][cl]);
                if (at >= 0) *reinterpret_cast<float4*>(A + (jj + at) * lda + jj + cl) = v;
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (pos[q] >= 0) {
                float* rp = A + (jj + pos[q]) * lda + jj;
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (k < w) rp[k] = x[q][k];
            }
    }
}

// The rest of the panel below a factored sub-panel [jj, jj + W):
// A[r, c] -= sum_k L21[r, k] U12[k, c] for the `below` rows from jj + W and
// columns [jj + W, c1), summed over k in order by fused multiply-adds.  One
// thread per row and group of 8 columns (threads of one row adjacent, so a
// row's groups are read and written together).  vec: A's rows 16-byte
// aligned at these columns.  The next sub-panel's W columns also go to next
// (rows x W) if there is one.
template <int W>
__global__ __launch_bounds__(256) void lu_sub_update(float* A, int64_t lda, int64_t jj, int below, int64_t c1, int vec,
                                                     float* next) {
    __shared__ __attribute__((aligned(16))) float U[W][kNb];
    const int cols = (int)(c1 - jj - W);  // 1 .. kNb - W
    constexpr int kPer = W * kNb / 256;
    float uv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = threadIdx.x + 256 * u, c = e % kNb;
        uv[u] = A[(jj + e / kNb) * lda + jj + W + (c < cols ? c : 0)];
    }
    const uint32_t groups = (uint32_t)(cols + 7) / 8, t = blockIdx.x * 256u + threadIdx.x;
    const int row = (int)(t / groups), cg = (int)(t % groups) * 8, r = min(row, below - 1);
    const int nc = cols - cg < 8 ? cols - cg : 8;
    float* rp = A + (jj + W + r) * lda + jj;
    float* cp = rp + W + cg;
    float l[W], acc[8];
    if (vec) {
#pragma unroll
        for (int k = 0; k < W; k += 4) {
            const float4 v = *reinterpret_cast<const float4*>(rp + k);
            l[k] = v.x, l[k + 1] = v.y, l[k + 2] = v.z, l[k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < W; ++k) l[k] = rp[k];
    }
    if (vec && nc == 8) {
        const float4 a0 = reinterpret_cast<const float4*>(cp)[0], a1 = reinterpret_cast<const float4*>(cp)[1];
        acc[0] = a0.x, acc[1] = a0.y, acc[2] = a0.z, acc[3] = a0.w;
        acc[4] = a1.x, acc[5] = a1.y, acc[6] = a1.z, acc[7] = a1.w;
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = c < nc ? cp[c] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = threadIdx.x + 256 * u;
        U[e / kNb][e % kNb] = uv[u];
    }
    __syncthreads();
    if (row >= below) return;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const float4 u0 = *reinterpret_cast<const float4*>(&U[k][cg]), u1 = *reinterpret_cast<const float4*>(&U[k][cg + 4]);
        const float u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = __builtin_fmaf(-l[k], u[c], acc[c]);
    }
    if (vec && nc == 8) {
        reinterpret_cast<float4*>(cp)[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        reinterpret_cast<float4*>(cp)[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (c < nc) cp[c] = acc[c];
    }
    if (next != nullptr && cg < W) {  // (entries past nc: never read)
        float4* np = reinterpret_cast<float4*>(next + (int64_t)row * W + cg);
        np[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        np[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
}

// The first sub-panel's columns A[j : j + rows, j : j + W] as rows x W (those
// past the matrix left out).  One thread per row and 8 columns.
template <int W>
__global__ __launch_bounds__(256) void lu_sub_gather(int rows, const float* A, int64_t lda, int64_t j, int w, int vec,
                                                     float* next) {
    const int t = blockIdx.x * 256 + threadIdx.x, r = t / (W / 8), c0 = t % (W / 8) * 8;
    if (r >= rows || c0 >= w) return;
    const float* rp = A + (j + r) * lda + j + c0;
    float* np = next + (int64_t)r * W + c0;
    if (vec && c0 + 8 <= w) {
        reinterpret_cast<float4*>(np)[0] = reinterpret_cast<const float4*>(rp)[0];
        reinterpret_cast<float4*>(np)[1] = reinterpret_cast<const float4*>(rp)[1];
    } else {
        for (int c = 0; c < 8 && c0 + c < w; ++c) np[c] = rp[c];
    }
}

// The panel's row moves on every column outside it and, right of it, the
// block row solved with the panel's unit lower triangle (U12 = L11^-1 A12),
// 64 columns per workgroup.  The moved rows of a column are all loaded (64-float row
// pieces, all in flight) before any is stored.  The solve has four lanes
// per column, lane p holding rows i = p mod 4 (of kNb, in registers); unknown
// k reaches the quad by DPP, and the rows below it take their multiply-add:
// the same operations in the same order per element as one thread per
// column.  12 us per panel at n = 2048 against 5.2 + 13.7 us for the
// exchanges one after the other and a thread per column.
constexpr int kTStride = kNb + 16;  // rows 16 banks apart: the quads' reads of a column do not collide
template <int K4>
__device__ __forceinline__ float quad_lane(float v) {  // lane K4 of each quad, to all four
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), K4 * 0x55, 0xF, 0xF, false));
}
__global__ __launch_bounds__(256) void lu_moves_trsm(int64_t n, float* A, int64_t lda, int64_t j, int w,
                                                     const LuMoves* moves) {
    __shared__ __attribute__((aligned(16))) float LT[kNb][4][kNb / 4];  // [k][p][m]: L11[4 m + p][k]
    __shared__ float T[kNb * kTStride];
    const int tid = threadIdx.x;
    const int64_t nleft = (j + kNb - 1) / kNb;  // workgroups of columns before the panel
    const bool right = blockIdx.x >= nleft;
    const int64_t c0 = right ? j + w + (blockIdx.x - nleft) * kNb : (int64_t)blockIdx.x * kNb;
    const int64_t cend = right ? n : j;
    const int col = tid & (kNb - 1), r0 = tid / kNb;
    const bool mine = c0 + col < cend;
    // the moves by way of LDS and no branch around a load, so that all of a
    // thread's rows are in flight together
    __shared__ int from[2 * kNb], to[2 * kNb];
    const int nm = w + moves->ndisp;
    if (tid < 2 * kNb) {
        const int d = min(max(tid - w, 0), kNb - 1), t = min(tid, kNb - 1);
        const int top = moves->top[t], src = moves->src[d], dst = moves->dst[d];
        from[tid] = tid >= nm ? 0 : tid < w ? top : src;
        to[tid] = tid >= nm ? 0 : tid < w ? tid : dst;
    }
    __syncthreads();
    float* cp = A + j * lda + c0 + col;
    const float* lp = mine ? cp : A + j * lda + c0;
    constexpr int kPer = 2 * kNb * kNb / 256;
    float v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[u] = lp[(int64_t)from[r0 + 4 * u] * lda];
    if (right) {  // (then w == kNb)
        float lv[kNb * kNb / 256];
#pragma unroll
        for (int u = 0; u < kNb * kNb / 256; ++u) {
            const int e = tid + 256 * u;
            lv[u] = A[(j + e / kNb) * lda + j + e % kNb];
        }
#pragma unroll
        for (int u = 0; u < kNb * kNb / 256; ++u) {
            const int e = tid + 256 * u, i = e / kNb, k = e % kNb;
            LT[k][i & 3][i >> 2] = lv[u];
        }
    }
    memory_barrier();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int r = r0 + 4 * u;
        if (!mine || r >= nm) continue;
        if (right && r < w) T[r * kTStride + col] = v[u];
        else cp[(int64_t)to[r] * lda] = v[u];
    }
    if (!right) return;
    __syncthreads();
    const int p = tid & 3, sc = tid >> 2;  // this quad's column
    float x[kNb / 4];
#pragma unroll
    for (int m = 0; m < kNb / 4; ++m) x[m] = T[(4 * m + p) * kTStride + sc];
    auto unknown = [&](auto kcst) {
        constexpr int k = decltype(kcst)::value, m0 = k / 4, k4 = k % 4;
        const float xk = quad_lane<k4>(x[m0]);
        if constexpr (k4 < 3) {
            const float u = __builtin_fmaf(-LT[k][p][m0], xk, x[m0]);
            x[m0] = p > k4 ? u : x[m0];
        }
#pragma unroll
        for (int m = m0 + 1; m < kNb / 4; ++m) x[m] = __builtin_fmaf(-LT[k][p][m], xk, x[m]);
    };
    [&]<int... Ks>(std::integer_sequence<int, Ks...>) {
        (unknown(std::integral_constant<int, Ks>{}), ...);
    }(std::make_integer_sequence<int, kNb - 1>{});
#pragma unroll
    for (int m = 0; m < kNb / 4; ++m) T[(4 * m + p) * kTStride + sc] = x[m];
    __syncthreads();
    if (!mine) return;
#pragma unroll
    for (int u = 0; u < kNb / 4; ++u) {
        const int r = r0 + 4 * u;
        cp[(int64_t)r * lda] = T[r * kTStride + col];
    }
}

// Panels of 4097 .. 8192 rows: sub-panels of 8 columns, four launches each.
// (lu_sub with 8 columns took 35 us against 15.3 + 5 here, as its one
// workgroup also moves the rows back: LU of 8192 36.5 ms against 32.4.)
// A narrow panel A[j:n, j:j+w] (w <= 8), copied by lu_gather8 into the
// contiguous rows x 8 array W, held in registers for all of its columns:
// thread t owns panel rows i = t + kP8Threads q (row j + i), q < kP8Rows (so
// rows = n - j <= kP8Threads kP8Rows).  One barrier per column c:
//   - each wavefront finds its largest |value| among its rows at or below the
//     diagonal (first row on ties; value and row then packed in one key); lane 0
//     writes the key and the lane owning that row the row's values to the
//     wavefront's LDS slot, and thread c (owner of the diagonal row, q = 0)
//     writes that row;
//   - after the barrier every thread reduces the slots by the same rule, so
//     each knows the pivot row p and both rows to exchange; their owners swap
//     them in registers, and every owned row below the diagonal is scaled by
//     the pivot and gets the rank-1 update of the columns to its right.
// The slots alternate between two LDS buffers by column parity: a buffer is
// written again two columns later, by threads that passed the barrier of the
// column in between, which every thread reaches only after reading it.  Rows
// move in and out of W as two 16-byte pieces; lu_subpanel_post writes the
// factored columns back.  Same arithmetic, operation by operation, as lu_panel.
constexpr int kP8 = 8, kP8Threads = 512, kP8Rows = 16, kP8Waves = kP8Threads / 64;

// Pivot candidates as one 64-bit key: the bits of |value| (non-negative
// floats order as their bit patterns) above the complement of the row, so
// the larger value wins and the lower row on ties in one unsigned compare;
// 0 is "no candidate" (a NaN, a row above the diagonal or past the matrix).
using P8Key = unsigned long long;
__device__ __forceinline__ P8Key p8_key(float a, int i) {
    return ((P8Key)__builtin_bit_cast(uint32_t, a) << 32) | (P8Key)(~(uint32_t)i);
}

// One step of the key max across lanes: the partner lane given by the DPP
// control CTRL.
template <int CTRL>
__device__ __forceinline__ void p8_dpp_max(P8Key& k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)k, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(k >> 32), CTRL, 0xF, 0xF, false);
    const P8Key o = ((P8Key)hi << 32) | lo;
    k = o > k ? o : k;
}

__device__ __forceinline__ P8Key p8_lane_key(P8Key k, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(k >> 32), lane);
    return ((P8Key)hi << 32) | lo;
}

__global__ __launch_bounds__(kP8Threads) void lu_panel8(int rows, float* W, int64_t j, int w, int32_t* ipiv,
                                                       int32_t* info) {
    __shared__ P8Key skey[2][kP8Waves];
    __shared__ __attribute__((aligned(16))) float srow[2][kP8Waves][kP8];
    __shared__ __attribute__((aligned(16))) float sdiag[2][kP8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float x[kP8Rows][kP8];
#pragma unroll
    for (int q = 0; q < kP8Rows; ++q) {
        const int i = tid + kP8Threads * q;
        float4 u = make_float4(0.0f, 0.0f, 0.0f, 0.0f), v = u;
        if (i < rows) {
            const float4* rp = reinterpret_cast<const float4*>(W + (int64_t)i * kP8);
            u = rp[0], v = rp[1];
        }
        x[q][0] = u.x, x[q][1] = u.y, x[q][2] = u.z, x[q][3] = u.w;
        x[q][4] = v.x, x[q][5] = v.y, x[q][6] = v.z, x[q][7] = v.w;
    }
#pragma unroll
    for (int c = 0; c < kP8; ++c) {
        if (c >= w) break;
        const int buf = c & 1;
        // the thread's candidate: its largest |value| at or below the diagonal
        // (fmaxf ignores NaN; the row of slot 0 above the diagonal counts as
        // -1), then the first of its rows holding it; rows past the matrix
        // hold zeros and come after all real rows, so they are taken only
        // when the thread has no real candidate, and are then rejected
        const float v0 = tid >= c ? fabsf(x[0][c]) : -1.0f;
        float m = v0;
#pragma unroll
        for (int q = 1; q < kP8Rows; ++q) m = fmaxf(m, fabsf(x[q][c]));
        int qs = kP8Rows;
#pragma unroll
        for (int q = kP8Rows - 1; q > 0; --q) qs = fabsf(x[q][c]) == m ? q : qs;
        qs = v0 == m ? 0 : qs;
        const int is = tid + kP8Threads * qs;
        P8Key best = (qs < kP8Rows && is < rows && m >= 0.0f) ? p8_key(m, is) : 0;
        // wavefront reduction: DPP inside each 16-lane row (xor 1, xor 2,
        // rotate 4, rotate 8 cover the row), then the four rows by readlane
        p8_dpp_max<0xB1>(best);   // quad_perm [1,0,3,2]
        p8_dpp_max<0x4E>(best);   // quad_perm [2,3,0,1]
        p8_dpp_max<0x124>(best);  // row_ror 4
        p8_dpp_max<0x128>(best);  // row_ror 8
        P8Key wk = p8_lane_key(best, 0);
#pragma unroll
        for (int r = 1; r < 4; ++r) {
            const P8Key o = p8_lane_key(best, 16 * r);
            wk = o > wk ? o : wk;
        }
        // the wavefront's candidate key and the row's values, written by the
        // lane owning it (slot wi / kP8Threads, uniform)
        if (lane == 0) skey[buf][wave] = wk;
        const int wi = (int)~(uint32_t)wk;
        if (wk != 0 && (wi & (kP8Threads - 1)) == tid) {
#pragma unroll
            for (int q = 0; q < kP8Rows; ++q)
                if (q == wi / kP8Threads)
#pragma unroll
                    for (int cc = 0; cc < kP8; ++cc) srow[buf][wave][cc] = x[q][cc];
        }
        if (tid == c)
#pragma unroll
            for (int cc = 0; cc < kP8; ++cc) sdiag[buf][cc] = x[0][cc];
        __syncthreads();
        P8Key pk = skey[buf][0];
        int pw = 0;
#pragma unroll
        for (int q = 1; q < kP8Waves; ++q) {
            const P8Key o = skey[buf][q];
            if (o > pk) pk = o, pw = q;
        }
        int pi = (int)~(uint32_t)pk;
        if (pk == 0) pi = c, pw = -1;  // no candidate (every |value| NaN): the diagonal row
        pi = __builtin_amdgcn_readfirstlane(pi);
        pw = __builtin_amdgcn_readfirstlane(pw);
        // both rows read whole and at once (one LDS round trip), then chosen
        const float4* dp = reinterpret_cast<const float4*>(sdiag[buf]);
        const float4* sp = reinterpret_cast<const float4*>(srow[buf][pw >= 0 ? pw : 0]);
        const float4 d0 = dp[0], d1 = dp[1], s0 = sp[0], s1 = sp[1];
        const float dr[kP8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        const float sr[kP8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        float pr[kP8];
#pragma unroll
        for (int cc = 0; cc < kP8; ++cc) pr[cc] = pw >= 0 ? sr[cc] : dr[cc];
        if (tid == 0) ipiv[j + c] = (int32_t)(j + pi);
        if (pi != c) {  // two lanes exchange rows j + c (slot 0 of thread c) and j + pi
            if (tid == (pi & (kP8Threads - 1))) {
#pragma unroll
                for (int q = 0; q < kP8Rows; ++q)
                    if (q == pi / kP8Threads)
#pragma unroll
                        for (int cc = 0; cc < kP8; ++cc) x[q][cc] = dr[cc];
            }
            if (tid == c)
#pragma unroll
                for (int cc = 0; cc < kP8; ++cc) x[0][cc] = pr[cc];
        }
        const float pv = pr[c];  // the pivot row is now row j + c
        if (tid == 0 && pv == 0.0f && *info == 0) *info = (int32_t)(j + c + 1);
        if (pv != 0.0f) {
            // rows below the diagonal; rows past the matrix hold zeros, take the
            // update harmlessly (or skip it with their wavefront) and are never
            // stored or chosen as pivots
            const float rp = 1.0f / pv;
#pragma unroll
            for (int q = 0; q < kP8Rows; ++q) {
                if (kP8Threads * q + 64 * wave >= rows) continue;  // the wavefront's rows of slot q are all past the matrix
                const bool below = q > 0 || tid > c;
                const float l = x[q][c] * rp;
                x[q][c] = below ? l : x[q][c];
#pragma unroll
                for (int cc = c + 1; cc < kP8; ++cc) {
                    const float u = __builtin_fmaf(-l, pr[cc], x[q][cc]);
                    x[q][cc] = below ? u : x[q][cc];
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kP8Rows; ++q) {
        const int i = tid + kP8Threads * q;
        if (i < rows) {
            float4* rp = reinterpret_cast<float4*>(W + (int64_t)i * kP8);
            rp[0] = make_float4(x[q][0], x[q][1], x[q][2], x[q][3]);
            rp[1] = make_float4(x[q][4], x[q][5], x[q][6], x[q][7]);
        }
    }
}

// The sub-panel A[j:j+rows, j:j+w] (w <= kP8) copied into W (rows x kP8,
// row-major, 16-byte aligned; columns from w on zero), one thread per row
// over as many workgroups as it takes (lu_subpanel_post writes it back the
// same way): A's rows are lda apart, and one workgroup fetching them all
// (each row a separate line and page) took most of the panel kernel's time.
// vec: w == kP8 and A's rows 16-byte aligned at column j (two 16-byte pieces
// per row), else element by element.
__global__ __launch_bounds__(256) void lu_gather8(const float* A, int64_t lda, int64_t j, int rows, int w, int vec,
                                                  float* W) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= rows) return;
    const float* rp = A + (j + i) * lda + j;
    float4* wp = reinterpret_cast<float4*>(W + (int64_t)i * kP8);
    if (vec) {
        wp[0] = *reinterpret_cast<const float4*>(rp);
        wp[1] = *reinterpret_cast<const float4*>(rp + 4);
    } else {
        float v[kP8];
#pragma unroll
        for (int c = 0; c < kP8; ++c) v[c] = c < w ? rp[c] : 0.0f;
        wp[0] = make_float4(v[0], v[1], v[2], v[3]);
        wp[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// After lu_panel8 on the sub-panel at column jj of the panel [c0, c1):
// blocks 0 .. nb-1 write the factored sub-panel back from W, one thread per
// row (as lu_gather8 read it); block nb gives each column of the panel
// outside the sub-panel one thread, which applies the sub-panel's row swaps
// to its column in order and, right of the sub-panel, solves the 8 rows jj ..
// jj+7 of its column with the unit lower block L11 (U12 = L11^-1 A12, L11
// from W).  The columns are independent, so swaps and solve need no barrier
// between them, and the write-back touches none of their elements.
__global__ __launch_bounds__(256) void lu_subpanel_post(float* A, int64_t lda, int64_t jj, int rows, int wi, int vec,
                                                        const float* W, const int32_t* ipiv, int64_t c0, int64_t c1,
                                                        int nb) {
    if ((int)blockIdx.x < nb) {
        const int i = blockIdx.x * 256 + threadIdx.x;
        if (i >= rows) return;
        float* rp = A + (jj + i) * lda + jj;
        const float4* wp = reinterpret_cast<const float4*>(W + (int64_t)i * kP8);
        if (vec) {
            *reinterpret_cast<float4*>(rp) = wp[0];
            *reinterpret_cast<float4*>(rp + 4) = wp[1];
        } else {
            const float4 u = wp[0], v = wp[1];
            const float e[kP8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
            for (int c = 0; c < kP8; ++c)
                if (c < wi) rp[c] = e[c];
        }
        return;
    }
    __shared__ float L[kP8][kP8];
    if (threadIdx.x < kP8 * kP8) L[threadIdx.x / kP8][threadIdx.x % kP8] = W[threadIdx.x];
    __syncthreads();
    const int64_t col = c0 + threadIdx.x;  // c1 - c0 <= kNb < 256
    if (col >= c1 || (col >= jj && col < jj + wi)) return;
    for (int c = 0; c < wi; ++c) {
        const int64_t k = jj + c, p = ipiv[k];
        if (p != k) {
            const float t = A[k * lda + col];
            A[k * lda + col] = A[p * lda + col];
            A[p * lda + col] = t;
        }
    }
    if (col < jj + wi) return;  // left of the sub-panel: swaps only
    // right of it (then wi == kP8: only the panel's last sub-panel is narrower)
    float x[kP8];
#pragma unroll
    for (int i = 0; i < kP8; ++i) x[i] = A[(jj + i) * lda + col];
#pragma unroll
    for (int i = 1; i < kP8; ++i)
#pragma unroll
        for (int k = 0; k < i; ++k) x[i] = __builtin_fmaf(-L[i][k], x[k], x[i]);
#pragma unroll
    for (int i = 0; i < kP8; ++i) A[(jj + i) * lda + col] = x[i];
}

// The rest of the panel after a factored sub-panel [jj, jj + 8): A[r, c] -=
// sum_k L21[r, k] U12[k, c] for rows r in [jj + 8, jj + 8 + below) and
// columns c in [jj + 8, c1), L21 from the sub-panel's copy W (its rows from 8
// on) and U12 = A[jj:jj+8, c] (solved by lu_subpanel_post), summed over k in
// order by fused multiply-adds.  One thread per row and group of 8 columns
// (threads of one row adjacent, so a row's groups are read and written
// together).  The first group is the next sub-panel: its updated values also
// go to that sub-panel's copy Wn (row r at r - jj - 8, columns from wn on
// zero), so it needs no gather.  vec: A's rows 16-byte aligned at these
// columns.
__global__ __launch_bounds__(256) void lu_subpanel_update(float* A, int64_t lda, int64_t jj, int below, int64_t c1,
                                                          const float* W, float* Wn, int wn, int vec) {
    __shared__ float U[kP8][kNb];
    const int cols = (int)(c1 - jj - kP8);  // 1 .. kNb - kP8
    for (int e = threadIdx.x; e < kP8 * cols; e += 256) U[e / cols][e % cols] = A[(jj + e / cols) * lda + jj + kP8 + e % cols];
    __syncthreads();
    const int groups = (cols + kP8 - 1) / kP8;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = (int)(t / groups), g = (int)(t % groups);
    if (r >= below) return;
    const int cg = g * kP8;                          // first column of the group, from jj + 8
    const int nc = cols - cg < kP8 ? cols - cg : kP8;  // columns in the group
    const float4* lp = reinterpret_cast<const float4*>(W + (int64_t)(kP8 + r) * kP8);
    const float4 l0 = lp[0], l1 = lp[1];
    const float l[kP8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
    float* cp = A + (jj + kP8 + r) * lda + jj + kP8 + cg;
    float acc[kP8];
    if (vec && nc == kP8) {
        const float4 a0 = reinterpret_cast<const float4*>(cp)[0], a1 = reinterpret_cast<const float4*>(cp)[1];
        acc[0] = a0.x, acc[1] = a0.y, acc[2] = a0.z, acc[3] = a0.w;
        acc[4] = a1.x, acc[5] = a1.y, acc[6] = a1.z, acc[7] = a1.w;
    } else {
#pragma unroll
        for (int cc = 0; cc < kP8; ++cc) acc[cc] = cc < nc ? cp[cc] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kP8; ++k)
#pragma unroll
        for (int cc = 0; cc < kP8; ++cc)
            if (cc < nc) acc[cc] = __builtin_fmaf(-l[k], U[k][cg + cc], acc[cc]);
    if (vec && nc == kP8) {
        reinterpret_cast<float4*>(cp)[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        reinterpret_cast<float4*>(cp)[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    } else {
#pragma unroll
        for (int cc = 0; cc < kP8; ++cc)
            if (cc < nc) cp[cc] = acc[cc];
    }
    if (g == 0) {
        float4* wp = reinterpret_cast<float4*>(Wn + (int64_t)r * kP8);
        float v[kP8];
#pragma unroll
        for (int cc = 0; cc < kP8; ++cc) v[cc] = cc < wn ? acc[cc] : 0.0f;
        wp[0] = make_float4(v[0], v[1], v[2], v[3]);
        wp[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// The panel's row swaps (rows j .. j+w-1 with ipiv[.]) on every column
// outside the panel, one thread per column, swaps in order.
__global__ __launch_bounds__(256) void lu_laswp(int64_t n, float* A, int64_t lda, int64_t j, int w,
                                                const int32_t* ipiv) {
    const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (col >= n || (col >= j && col < j + w)) return;
    for (int c = 0; c < w; ++c) {
        const int64_t k = j + c, p = ipiv[k];
        if (p != k) {
            const float t = A[k * lda + col];
            A[k * lda + col] = A[p * lda + col];
            A[p * lda + col] = t;
        }
    }
}

// U12 = L11^-1 A12 for the block row A[j:j+kNb, j+kNb:n] (L11 unit lower,
// kept in LDS), one thread per column, the column in registers.  L11 comes
// in as 16 loads per thread issued together, then 16 LDS stores (stored as
// each arrived, the loads went out one latency at a time); every lane reads
// the same entries, four per LDS read, and the multiply-adds run in the same
// order as one entry at a time.
__global__ __launch_bounds__(256) void lu_trsm(int64_t n, float* A, int64_t lda, int64_t j) {
    __shared__ __attribute__((aligned(16))) float L[kNb][kNb];
    constexpr int kPer = kNb * kNb / 256;
    float lv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = threadIdx.x + 256 * u;
        lv[u] = A[(j + e / kNb) * lda + j + e % kNb];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = threadIdx.x + 256 * u;
        L[e / kNb][e % kNb] = lv[u];
    }
    __syncthreads();
    const int64_t col = j + kNb + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (col >= n) return;
    float x[kNb];
#pragma unroll
    for (int i = 0; i < kNb; ++i) x[i] = A[(j + i) * lda + col];
#pragma unroll
    for (int i = 1; i < kNb; ++i)
#pragma unroll
        for (int k4 = 0; k4 < i; k4 += 4) {
            const float4 l = *reinterpret_cast<const float4*>(&L[i][k4]);
            const float lk[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
            for (int k = k4; k < k4 + 4 && k < i; ++k) x[i] = __builtin_fmaf(-lk[k - k4], x[k], x[i]);
        }
#pragma unroll
    for (int i = 0; i < kNb; ++i) A[(j + i) * lda + col] = x[i];
}

// Diagonal block [s, s+w) of the factors solved for the right-hand sides
// V[s:s+w, 0:nrhs] in place: unit lower (forward) or upper (backward, with
// the diagonal).  One wavefront per right-hand side, lane i holding row i:
// the lane's row of the block is loaded into registers once (every load in
// flight together), and each finished unknown reaches the other lanes by
// readlane, so the w dependent steps wait on no memory and no barrier.
static_assert(kNb == 64, "one wavefront per diagonal block");
template <bool LOWER>
__global__ __launch_bounds__(kNb) void lu_trsv_block(const float* LU, int64_t ldlu, int64_t s, int w, float* V,
                                                     int64_t ldv) {
    const int i = threadIdx.x;
    const int64_t q = blockIdx.x;
    const float* row = LU + (s + (i < w ? i : 0)) * ldlu + s;
    float r[kNb];
#pragma unroll
    for (int k = 0; k < kNb; ++k) r[k] = k < w ? row[k] : 0.0f;
    float xi = i < w ? V[(s + i) * ldv + q] : 0.0f;
    auto lane_value = [](float v, int k) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
    };
    if constexpr (LOWER) {
#pragma unroll
        for (int k = 0; k < kNb; ++k) {
            if (k < w) {
                const float xk = lane_value(xi, k);
                if (i > k && i < w) xi = __builtin_fmaf(-r[k], xk, xi);
            }
        }
    } else {
#pragma unroll
        for (int k = kNb - 1; k >= 0; --k) {
            if (k < w) {
                if (i == k) xi = xi / r[k];
                const float xk = lane_value(xi, k);
                if (i < k) xi = __builtin_fmaf(-r[k], xk, xi);
            }
        }
    }
    if (i < w) V[(s + i) * ldv + q] = xi;
}

// A whole substitution (forward with the unit lower triangle, or backward
// with the upper one) of nrhs right-hand sides in one launch, in place in V.
// One wavefront per block of kNb rows and R right-hand sides, lane i holding
// row i: as each block before it is published, it takes that block's
// multiply-adds (its 64 entries of the row, loaded ahead of the wait, times the
// solved unknowns, by readlane, in column order); then it solves its diagonal
// block as lu_trsv_block does and publishes its unknowns.  The same
// operations in the same order per element for any R, and as one launch per
// block.
// Bound by the chain from block to block: a publication seen, 64 multiply-adds,
// the 64 dependent steps of the diagonal block.  At n = 2048, one right-hand
// side, 102 us forward and 148 backward against 32 launches of 7.8 and 9.1 us.
// R = 2 and 4 where the wavefronts of R = 1 would come in many turns: the rows'
// entries are then loaded once for them (chain_rhs).
//
// A published unknown is one 64-bit word, its value beside the launch's tag,
// stored and polled as a relaxed agent-scope atomic, so the value needs no
// ordering against a flag.  Z (n x nrhs words) starts as zeros, tags count up
// from 1.  The blocks are taken in order from a ticket counter (`first`: the
// tickets of the launches before), so a wavefront waits only for blocks whose
// wavefronts already run: every wait ends.
template <bool LOWER, int R>
__global__ __launch_bounds__(kNb) void lu_chain(const float* LU, int64_t ldlu, int64_t n, int64_t nrhs, int nblk,
                                                float* V, int64_t ldv, unsigned long long* Z, uint32_t tag,
                                                uint32_t* ticket, uint32_t first, int vec) {
    const int i = threadIdx.x;
    uint32_t id = 0;
    if (i == 0) id = atomicAdd(ticket, 1u) - first;
    id = (uint32_t)__builtin_amdgcn_readfirstlane((int)id);
    const uint32_t groups = (uint32_t)((nrhs + R - 1) / R);
    const int b = (int)(id / groups);
    const int64_t q0 = (int64_t)(id % groups) * R;
    const int blk = LOWER ? b : nblk - 1 - b;
    const int64_t s = (int64_t)blk * kNb;
    const int w = (int)min(n - s, (int64_t)kNb);
    const float* row = LU + (s + (i < w ? i : 0)) * ldlu;
    auto load = [&](int64_t c0, int cw, float (&d)[kNb]) {  // the row's entries of columns c0 ..
        if (vec && cw == kNb) {
#pragma unroll
            for (int k = 0; k < kNb; k += 4) {
                const float4 v = *reinterpret_cast<const float4*>(row + c0 + k);
                d[k] = v.x, d[k + 1] = v.y, d[k + 2] = v.z, d[k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < kNb; ++k) d[k] = k < cw ? row[c0 + k] : 0.0f;
        }
    };
    // (past the last right-hand side: the last one again, not stored)
    auto rhs = [&](int r) { return R == 1 ? q0 : min(q0 + r, nrhs - 1); };
    float d[kNb], x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = i < w ? V[(s + i) * ldv + rhs(r)] : 0.0f;
    load(s, w, d);  // the diagonal block
    for (int t = 0; t < b; ++t) {
        const int kb = LOWER ? t : nblk - 1 - t;
        const int64_t c0 = (int64_t)kb * kNb;
        const int cw = (int)min(n - c0, (int64_t)kNb);
        float l[kNb], u[R];
        load(c0, cw, l);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned long long* z = Z + rhs(r) * n + c0;
            unsigned long long v = 0;
            for (;;) {
                if (i < cw) v = __hip_atomic_load(z + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__all(i >= cw || (uint32_t)(v >> 32) == tag)) break;
                __builtin_amdgcn_s_sleep(1);
            }
            u[r] = __builtin_bit_cast(float, (uint32_t)v);
        }
        if (cw == kNb) {
#pragma unroll
            for (int k = 0; k < kNb; ++k)
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = __builtin_fmaf(-l[k], lane_of(u[r], k), x[r]);
        } else {
#pragma unroll
            for (int k = 0; k < kNb; ++k)
                if (k < cw)
#pragma unroll
                    for (int r = 0; r < R; ++r) x[r] = __builtin_fmaf(-l[k], lane_of(u[r], k), x[r]);
        }
    }
    if constexpr (LOWER) {
#pragma unroll
        for (int k = 0; k < kNb; ++k)
            if (k < w)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float xk = lane_of(x[r], k);
                    if (i > k && i < w) x[r] = __builtin_fmaf(-d[k], xk, x[r]);
                }
    } else {
#pragma unroll
        for (int k = kNb - 1; k >= 0; --k)
            if (k < w)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (i == k) x[r] = x[r] / d[k];
                    const float xk = lane_of(x[r], k);
                    if (i < k) x[r] = __builtin_fmaf(-d[k], xk, x[r]);
                }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t q = q0 + r;
        if (i >= w || q >= nrhs) continue;
        const unsigned long long word = ((unsigned long long)tag << 32) | __builtin_bit_cast(uint32_t, x[r]);
        __hip_atomic_store(Z + q * n + s + i, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        V[(s + i) * ldv + q] = x[r];
    }
}

// One block step of the substitution, for right-hand side q = blockIdx.y:
// the diagonal block [s, s+w) of the factors solved (unit lower, forward, or
// upper with the diagonal, backward) from In[s:s+w, q] by the first
// wavefront of every workgroup, as in lu_trsv_block (each workgroup solves
// the same small system, so none waits for another); workgroup 0 writes the
// solution to Out[s:s+w, q]; and the rows still to be solved (forward: below
// the block, backward: above it), one per thread, are updated in place,
// In[r, q] -= LU[r, s:s+w] . x, by multiply-adds in column order.  In and
// Out are distinct arrays, so no workgroup overwrites right-hand sides
// another still reads.  vec: LU's rows 16-byte aligned at column s.
template <bool LOWER>
__global__ __launch_bounds__(256) void lu_subst_step(const float* LU, int64_t ldlu, int64_t n, int64_t s, int w,
                                                     float* In, int64_t ldi, float* Out, int64_t ldo, int vec) {
    __shared__ float xs[kNb];
    const int64_t q = blockIdx.y;
    if (threadIdx.x < kNb) {
        const int i = threadIdx.x;
        const float* row = LU + (s + (i < w ? i : 0)) * ldlu + s;
        float r[kNb];
#pragma unroll
        for (int k = 0; k < kNb; ++k) r[k] = k < w ? row[k] : 0.0f;
        float xi = i < w ? In[(s + i) * ldi + q] : 0.0f;
        auto lane_value = [](float v, int k) {
            return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
        };
        if constexpr (LOWER) {
#pragma unroll
            for (int k = 0; k < kNb; ++k) {
                if (k < w) {
                    const float xk = lane_value(xi, k);
                    if (i > k && i < w) xi = __builtin_fmaf(-r[k], xk, xi);
                }
            }
        } else {
#pragma unroll
            for (int k = kNb - 1; k >= 0; --k) {
                if (k < w) {
                    if (i == k) xi = xi / r[k];
                    const float xk = lane_value(xi, k);
                    if (i < k) xi = __builtin_fmaf(-r[k], xk, xi);
                }
            }
        }
        xs[i] = xi;  // 0 for i >= w
        if (blockIdx.x == 0 && i < w) Out[(s + i) * ldo + q] = xi;
    }
    __syncthreads();
    const int64_t r0 = LOWER ? s + w : 0, r1 = LOWER ? n : s;
    const int64_t rr = r0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (rr >= r1) return;
    const float* lr = LU + rr * ldlu + s;
    float acc = In[rr * ldi + q];
    if (vec && w == kNb) {
#pragma unroll
        for (int k4 = 0; k4 < kNb / 4; ++k4) {
            const float4 a = reinterpret_cast<const float4*>(lr)[k4];
            acc = __builtin_fmaf(-a.x, xs[4 * k4], acc);
            acc = __builtin_fmaf(-a.y, xs[4 * k4 + 1], acc);
            acc = __builtin_fmaf(-a.z, xs[4 * k4 + 2], acc);
            acc = __builtin_fmaf(-a.w, xs[4 * k4 + 3], acc);
        }
    } else {
        for (int k = 0; k < w; ++k) acc = __builtin_fmaf(-lr[k], xs[k], acc);
    }
    In[rr * ldi + q] = acc;
}

// dst[i, :] = src[perm[i], :] (rows of nrhs FP32 values); and zeros into the
// first `words` <= n x nrhs + 1 of Z.
__global__ __launch_bounds__(256) void gather_rows(int64_t n, int64_t nrhs, const int32_t* perm, const float* src,
                                                   int64_t lds, float* dst, int64_t ldd, unsigned long long* Z,
                                                   int64_t words) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e + 1 < words) Z[e + 1] = 0;
    if (e == 0 && words > 0) Z[0] = 0;
    if (e >= n * nrhs) return;
    const int64_t i = e / nrhs, q = e % nrhs;
    dst[i * ldd + q] = src[(int64_t)perm[i] * lds + q];
}

__global__ __launch_bounds__(256) void f64_to_f32(int64_t rows, int64_t cols, const double* X, int64_t ldx, float* Y,
                                                  int64_t ldy) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= rows * cols) return;
    const int64_t i = e / cols, q = e % cols;
    Y[i * ldy + q] = (float)X[i * ldx + q];
}

// X = D (first) or X += D, X FP64, D FP32.
__global__ __launch_bounds__(256) void accumulate_f64(int64_t rows, int64_t cols, const float* D, int64_t ldd,
                                                      double* X, int64_t ldx, int first) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= rows * cols) return;
    const int64_t i = e / cols, q = e % cols;
    const double d = (double)D[i * ldd + q];
    X[i * ldx + q] = first ? d : X[i * ldx + q] + d;
}

// R = B - A X in FP64: one wavefront per (row, right-hand side), lanes over K.
__global__ __launch_bounds__(256) void residual_f64(int64_t n, int64_t nrhs, const double* A, int64_t lda,
                                                   const double* X, int64_t ldx, const double* B, int64_t ldb,
                                                   double* R, int64_t ldr) {
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (w >= n * nrhs) return;
    const int64_t i = w / nrhs, q = w % nrhs;
    double acc = 0.0;
    for (int64_t k = lane; k < n; k += 64) acc = fma(A[i * lda + k], X[k * ldx + q], acc);
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) R[i * ldr + q] = B[i * ldb + q] - acc;
}

// Row sums of |A| (FP64), one wavefront per row.
__global__ __launch_bounds__(256) void abs_row_sums(int64_t n, const double* A, int64_t lda, double* out) {
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= n) return;
    double acc = 0.0;
    for (int64_t k = lane; k < n; k += 64) acc += fabs(A[i * lda + k]);
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) out[i] = acc;
}

// out[q] = max_i |V[i, q]| for each of the nrhs columns of V (one workgroup
// per column); with rows_only (nrhs = 1 of a vector v), the max of v.
__global__ __launch_bounds__(256) void col_abs_max(int64_t n, int64_t nrhs, const double* V, int64_t ldv,
                                                   double* out) {
    __shared__ double red[256];
    const int64_t q = blockIdx.x;
    double m = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) m = fmax(m, fabs(V[i * ldv + q]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[q] = red[0];
}

unsigned blocks(int64_t work, int per) { return (unsigned)std::max<int64_t>(1, (work + per - 1) / per); }

bool factor_mode_ok(int mode) {
    const int m = mode & MFG_MODE_MASK;
    return (mode & ~MFG_MODE_MASK) == 0 && m >= 0 && m < MFG_NUM_MODES;
}

}  // namespace

// Panels by height: up to kSubRows rows in sub-panels of 32 or 16 columns
// (lu_sub's registers hold the rows), up to kP8Threads x kP8Rows in sub-panels
// of 8 (lu_panel8), above that column by column (lu_panel).
constexpr int64_t kSubRows = 4096, kRows8 = (int64_t)kP8Threads * kP8Rows;
static int sub_width(int64_t rows) { return rows <= 2048 ? 32 : 16; }

// Floats of one copy of a sub-panel, and bytes of lu_factor_impl's device
// scratch: for lu_panel8 two copies of 8 columns (each at least the 8 x 8 diagonal
// block that lu_subpanel_post reads), over which, as one of 16, lu_sub's narrow
// sub-panels go once the rows left are few enough; the panel's row moves; the
// origin of each row.
static int64_t lu_copy_floats(int64_t n) { return n <= 2048 ? 0 : std::min(n, kRows8) * (n > kSubRows ? 8 : 16); }
static int64_t lu_copies(int64_t n) { return n > kSubRows ? 2 : 1; }
size_t lu_scratch_bytes(int64_t n) {
    return (size_t)(lu_copy_floats(n) * lu_copies(n)) * sizeof(float) + sizeof(LuMoves) + (size_t)n * sizeof(int32_t);
}

// One sub-panel by the workgroup whose registers hold its rows.
static int launch_lu_sub(int rows, const float* in, int64_t ldin, float* A, int64_t lda, int64_t j, int64_t jj, int w,
                         int cw, int vec, int32_t* ipiv, int32_t* info, int32_t* org, LuMoves* moves, int W,
                         hipStream_t s) {
#define MFG_LU_SUB(W_, Q_, NT_)                                                                                       \
    hipLaunchKernelGGL((lu_sub<W_, Q_, NT_>), dim3(1), dim3(NT_), 0, s, rows, in, ldin, A, lda, j, jj, w, cw, vec, ipiv, \
                       info, org, moves)
    if (W == 16) MFG_LU_SUB(16, 8, 512);
    else if (rows <= 512) MFG_LU_SUB(32, 2, 256);
    else if (rows <= 1024) MFG_LU_SUB(32, 4, 256);
    else MFG_LU_SUB(32, 4, 512);
#undef MFG_LU_SUB
    MFG_LAUNCH_CHECK();
    return MFG_OK;
}

// One panel [j, j + w) of at most kRows8 rows by sub-panels of 8 columns: each
// held in a contiguous copy (the first gathered by lu_gather8, the others
// written by the previous one's update; the two copies alternate), factored
// there in registers (lu_panel8), written back with its swaps applied across
// the panel and its block row solved (lu_subpanel_post), and the rest of the
// panel updated with K = 8 (lu_subpanel_update, L21 read from the copy).
static int lu_panel_by_8(int64_t n, float* A, int64_t lda, int64_t j, int w, int aligned, int32_t* ipiv, int32_t* info,
                         float* copy0, float* copy1, hipStream_t s) {
    float* const copies[2] = {copy0, copy1};
    int cur = 0;
    bool held = false;  // copies[cur] already holds this sub-panel
    for (int64_t jj = j; jj < j + w; jj += kP8) {
        const int wi = (int)std::min<int64_t>(kP8, j + w - jj);
        const int vec = wi == kP8 && aligned;
        const int rows = (int)(n - jj);
        float* const Wc = copies[cur];
        if (!held) {
            hipLaunchKernelGGL(lu_gather8, dim3(blocks(rows, 256)), dim3(256), 0, s, A, lda, jj, rows, wi, vec, Wc);
            MFG_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL(lu_panel8, dim3(1), dim3(kP8Threads), 0, s, rows, Wc, jj, wi, ipiv, info);
        MFG_LAUNCH_CHECK();
        const unsigned nb = blocks(rows, 256);
        hipLaunchKernelGGL(lu_subpanel_post, dim3(nb + 1), dim3(256), 0, s, A, lda, jj, rows, wi, vec, Wc, ipiv, j, j + w,
                           (int)nb);
        MFG_LAUNCH_CHECK();
        const int64_t right = j + w - (jj + wi);  // columns of the panel right of the sub-panel
        const int below = rows - wi;              // > 0 whenever right > 0 (then wi == kP8)
        held = right > 0 && below > 0;
        if (!held) continue;
        const int wn = (int)std::min<int64_t>(kP8, right);
        const int64_t threads = (int64_t)below * ((right + kP8 - 1) / kP8);
        hipLaunchKernelGGL(lu_subpanel_update, dim3(blocks(threads, 256)), dim3(256), 0, s, A, lda, jj, below, j + w, Wc,
                           copies[cur ^ 1], wn, aligned);
        MFG_LAUNCH_CHECK();
        cur ^= 1;
    }
    return MFG_OK;
}

// Blocked LU (see the file comment).  A, ipiv, info, scratch
// (lu_scratch_bytes(n)): device.  Per panel of 64 columns: its sub-panels
// (lu_sub), each followed by the update of the panel's columns right of it
// (lu_sub_update); the panel's row moves on all other columns and the block
// row's solve (lu_moves_trsm); the trailing update by mfg_gemm.  Sub-panels of
// 16 columns come from a copy rows x 16 written by the update before (the
// panel's first by lu_sub_gather): their rows are half of a 128-byte line, and
// what one CU can have outstanding is lines.  Taller panels, see kSubRows,
// swap their rows by lu_laswp and solve the block row by lu_trsm.
int lu_factor_impl(int64_t n, float* A, int64_t lda, int32_t* ipiv, int32_t* info, void* scratch, int mode,
                   hipStream_t s) {
    float* const copy = static_cast<float*>(scratch);
    LuMoves* const moves = reinterpret_cast<LuMoves*>(copy + lu_copy_floats(n) * lu_copies(n));
    int32_t* const org = reinterpret_cast<int32_t*>(moves + 1);
    const int vec = lda % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0;
    MFG_HIP_CHECK(hipMemsetAsync(info, 0, sizeof(int32_t), s));
    for (int64_t j = 0; j < n; j += kNb) {
        const int w = (int)std::min<int64_t>(kNb, n - j);
        const int64_t rest = n - j - w;  // > 0: then w == kNb
        if (n - j <= kSubRows) {
            const int W = sub_width(n - j);
            float* const next = W < 32 ? copy : nullptr;
            if (next != nullptr) {
                const int rows = (int)(n - j);
                if (W != 16 || (int64_t)rows * W > lu_copy_floats(n) * lu_copies(n)) return MFG_ERR_INTERNAL;
                hipLaunchKernelGGL(lu_sub_gather<16>, dim3(blocks((int64_t)rows * 2, 256)), dim3(256), 0, s, rows, A, lda, j,
                                   w, vec, next);
                MFG_LAUNCH_CHECK();
            }
            for (int64_t jj = j; jj < j + w; jj += W) {
                const int wi = (int)std::min<int64_t>(W, j + w - jj), rows = (int)(n - jj);
                const int st = launch_lu_sub(rows, next ? next : A + jj * lda + jj, next ? W : lda, A, lda, j, jj, wi, w,
                                             vec, ipiv, info, org, moves, W, s);
                if (st != MFG_OK) return st;
                const int64_t right = j + w - (jj + wi);  // columns of the panel right of the sub-panel (then wi == W)
                const int below = rows - wi;
                if (right <= 0 || below <= 0) continue;
                const dim3 g(blocks((int64_t)below * ((right + 7) / 8), 256)), t(256);
                if (W == 32) hipLaunchKernelGGL(lu_sub_update<32>, g, t, 0, s, A, lda, jj, below, j + w, vec, next);
                else hipLaunchKernelGGL(lu_sub_update<16>, g, t, 0, s, A, lda, jj, below, j + w, vec, next);
                MFG_LAUNCH_CHECK();
            }
            const unsigned g = (unsigned)((j + kNb - 1) / kNb + (rest + kNb - 1) / kNb);
            if (g > 0) {
                hipLaunchKernelGGL(lu_moves_trsm, dim3(g), dim3(256), 0, s, n, A, lda, j, w, moves);
                MFG_LAUNCH_CHECK();
            }
        } else {
            if (n - j <= kRows8) {
                if ((n - j) * 8 > lu_copy_floats(n) || lu_copies(n) < 2) return MFG_ERR_INTERNAL;
                const int st = lu_panel_by_8(n, A, lda, j, w, vec, ipiv, info, copy, copy + lu_copy_floats(n), s);
                if (st != MFG_OK) return st;
            } else {
                hipLaunchKernelGGL(lu_panel, dim3(1), dim3(kPanelThreads), 0, s, n, A, lda, j, w, ipiv, info);
                MFG_LAUNCH_CHECK();
            }
            hipLaunchKernelGGL(lu_laswp, dim3(blocks(n, 256)), dim3(256), 0, s, n, A, lda, j, w, ipiv);
            MFG_LAUNCH_CHECK();
            if (rest > 0) {
                hipLaunchKernelGGL(lu_trsm, dim3(blocks(rest, 256)), dim3(256), 0, s, n, A, lda, j);
                MFG_LAUNCH_CHECK();
            }
        }
        if (rest <= 0) continue;
        // A22 -= L21 U12 on the matrix cores, in the factorisation's mode
        float* a22 = A + (j + w) * lda + j + w;
        const int st = mfg_gemm(rest, rest, w, A + (j + w) * lda + j, lda, A + j * lda + j + w, lda, a22, lda, -1.0f,
                                1.0f, mode, (void*)s);
        if (st != MFG_OK) return st;
    }
    return MFG_OK;
}

// The row permutation of the sequential swaps in ipiv (device), on the host.
static int permutation(int64_t n, const int32_t* ipiv, std::vector<int32_t>& perm, hipStream_t s) {
    std::vector<int32_t> piv((size_t)n);
    MFG_HIP_CHECK(hipMemcpyAsync(piv.data(), ipiv, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, s));
    MFG_HIP_CHECK(hipStreamSynchronize(s));
    perm.resize((size_t)n);
    for (int64_t i = 0; i < n; ++i) perm[(size_t)i] = (int32_t)i;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t p = piv[(size_t)i];
        if (p < i || p >= n) return MFG_ERR_INVALID_ARG;  // not a pivot sequence of a factorisation
        std::swap(perm[(size_t)i], perm[(size_t)p]);
    }
    return MFG_OK;
}

// Device words of lu_chain (n x nrhs published unknowns and the ticket
// counter) and what its launches so far have used of them; none where
// lu_substitute does without.
struct ChainWords {
    unsigned long long* z = nullptr;
    uint32_t tag = 0, tickets = 0;
};
// Two blocks, the second not whole, and many right-hand sides: one launch per
// block (lu_subst_step); also of three, where only the words would take more
// than the 2 MB past which an allocation is 40 us.  us of mfg_lu_solve: n = 65
// with 400, 1000 and 3000 of them 71, 75, 103 against 75, 85, 144 of lu_chain,
// n = 100 74, 82, 121 and 78, 92, 152; n = 129 with 3000 175 and 212; but n = 128
// with 400 and 1000 85, 103 and 82, 97.
static bool subst_by_steps(int64_t n, int64_t nrhs) {
    if (n <= kNb || n >= 3 * kNb || nrhs > 65535) return false;
    return n < 2 * kNb ? nrhs > 300 : n * nrhs > (1 << 18) && n * nrhs <= (1 << 19);
}
static size_t chain_words(int64_t n, int64_t nrhs) {
    if (n <= kNb || nrhs > 65535 || n * nrhs > (int64_t)1 << 30 || subst_by_steps(n, nrhs)) return 0;
    return (size_t)(n * nrhs + 1);
}
// Right-hand sides per wavefront of lu_chain.  One wavefront's chain is the
// shortest with one of them; past the wavefronts that the chip holds, more share
// the loads of the factors, and all the earlier where rows are read an element
// at a time.  us of both substitutions with 1, 2 and 4, nrhs = 100, 400, 1000:
// n = 500 132 151 211, 228 214 259, 338 269 305; n = 2048 481 515 754, 1054 714
// 866, 2314 1335 1058; n = 777 239 219 308, 655 426 401, 1183 770 548; n = 2049
// 1185 650 773, 3667 1913 1207, 8708 4367 2261 (the last two odd; one launch per
// block of rows 302, 496, 944 and 947, 2299, 4679).
static int chain_rhs(int64_t nblk, int64_t nrhs, bool vec) {
    if (nrhs > std::min<int64_t>(vec ? 1200 : 700, (vec ? 22000 : 4500) / nblk)) return 4;
    return nrhs > std::min<int64_t>(vec ? 280 : 170, (vec ? 5500 : 1300) / nblk) ? 2 : 1;
}
// V = U^-1 L^-1 V (V: n x nrhs FP32, already permuted) in FP32, in place:
// with Y as large as scratch; forward and backward substitution by blocks of kNb
// rows, one launch each (lu_chain) or, without its words, one per block
// (lu_subst_step), with the same results.  One block of rows needs neither; beyond
// 65535 right-hand sides block by block: the diagonal block (lu_trsv_block), then
// the rest of V by an FP32 mfg_gemm.
static int lu_substitute(int64_t n, int64_t nrhs, const float* LU, int64_t ldlu, float* V, int64_t ldv, float* Y,
                         int64_t ldy, ChainWords& c, hipStream_t s) {
    const int64_t nblk = (n + kNb - 1) / kNb;
    const int vec = ldlu % 4 == 0 && reinterpret_cast<uintptr_t>(LU) % 16 == 0;
    if (c.z != nullptr) {
        const int R = chain_rhs(nblk, nrhs, vec != 0);
        const uint32_t grid = (uint32_t)(nblk * ((nrhs + R - 1) / R));
        uint32_t* ticket = reinterpret_cast<uint32_t*>(c.z + n * nrhs);
        for (int lower = 1; lower >= 0; --lower) {
            auto* kernel = lower ? (R == 4 ? lu_chain<true, 4> : R == 2 ? lu_chain<true, 2> : lu_chain<true, 1>)
                                 : (R == 4 ? lu_chain<false, 4> : R == 2 ? lu_chain<false, 2> : lu_chain<false, 1>);
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(kNb), 0, s, LU, ldlu, n, nrhs, (int)nblk, V, ldv, c.z, ++c.tag,
                               ticket, c.tickets, vec);
            MFG_LAUNCH_CHECK();
            c.tickets += grid;
        }
        return MFG_OK;
    }
    if (n > kNb && nrhs <= 65535) {
        for (int64_t b = 0; b < n; b += kNb) {  // forward, unit lower: V -> Y
            const int w = (int)std::min<int64_t>(kNb, n - b);
            hipLaunchKernelGGL(lu_subst_step<true>, dim3(blocks(n - b - w, 256), (unsigned)nrhs), dim3(256), 0, s, LU,
                               ldlu, n, b, w, V, ldv, Y, ldy, vec);
            MFG_LAUNCH_CHECK();
        }
        for (int64_t b = ((n - 1) / kNb) * kNb; b >= 0; b -= kNb) {  // backward, upper: Y -> V
            const int w = (int)std::min<int64_t>(kNb, n - b);
            hipLaunchKernelGGL(lu_subst_step<false>, dim3(blocks(b, 256), (unsigned)nrhs), dim3(256), 0, s, LU, ldlu, n,
                               b, w, Y, ldy, V, ldv, vec);
            MFG_LAUNCH_CHECK();
        }
        return MFG_OK;
    }
    const dim3 g((unsigned)nrhs);
    for (int64_t b = 0; b < n; b += kNb) {  // forward, unit lower
        const int w = (int)std::min<int64_t>(kNb, n - b);
        hipLaunchKernelGGL(lu_trsv_block<true>, g, dim3(kNb), 0, s, LU, ldlu, b, w, V, ldv);
        MFG_LAUNCH_CHECK();
        if (b + w < n) {
            const int st = mfg_gemm(n - b - w, nrhs, w, LU + (b + w) * ldlu + b, ldlu, V + b * ldv, ldv,
                                    V + (b + w) * ldv, ldv, -1.0f, 1.0f, MFG_F32, (void*)s);
            if (st != MFG_OK) return st;
        }
    }
    for (int64_t b = ((n - 1) / kNb) * kNb; b >= 0; b -= kNb) {  // backward, upper
        const int w = (int)std::min<int64_t>(kNb, n - b);
        hipLaunchKernelGGL(lu_trsv_block<false>, g, dim3(kNb), 0, s, LU, ldlu, b, w, V, ldv);
        MFG_LAUNCH_CHECK();
        if (b > 0) {
            const int st = mfg_gemm(b, nrhs, w, LU + b, ldlu, V + b * ldv, ldv, V, ldv, -1.0f, 1.0f, MFG_F32,
                                    (void*)s);
            if (st != MFG_OK) return st;
        }
    }
    return MFG_OK;
}

// X = (LU)^-1 P B with B, X n x nrhs FP32 (X may not alias B); B's contents are
// unspecified afterwards.  The chain's words are cleared the first time.
static int lu_solve_impl(int64_t n, int64_t nrhs, const float* LU, int64_t ldlu, const int32_t* dperm, float* B,
                         int64_t ldb, float* X, int64_t ldx, ChainWords& c, hipStream_t s) {
    const int64_t words = c.z != nullptr && c.tag == 0 ? (int64_t)chain_words(n, nrhs) : 0;
    hipLaunchKernelGGL(gather_rows, dim3(blocks(n * nrhs, 256)), dim3(256), 0, s, n, nrhs, dperm, B, ldb, X, ldx, c.z,
                       words);
    MFG_LAUNCH_CHECK();
    return lu_substitute(n, nrhs, LU, ldlu, X, ldx, B, ldb, c, s);
}

}  // namespace mfg

using namespace mfg;

namespace {

// Device buffers of one call, freed on every return path.
struct Buffers {
    std::vector<void*> ptrs;
    template <class T>
    int get(T** p, size_t count) {
        *p = nullptr;
        if (count == 0) count = 1;
        if (hipMalloc((void**)p, count * sizeof(T)) != hipSuccess) {
            (void)hipGetLastError();
            *p = nullptr;
            return MFG_ERR_NO_MEMORY;
        }
        ptrs.push_back(*p);
        return MFG_OK;
    }
    // `lead` bytes and, if there is memory for them, the chain's words.  One
    // allocation, as a second one and its free are 6 of the 55 us of a small
    // mfg_lu_solve; but two where that keeps the words within 2 MB, past which an
    // allocation is 40 us (n = 192, 1000 right-hand sides: 157 us with one, 120
    // with two).
    int get_with_chain(char** p, size_t lead, int64_t n, int64_t nrhs, ChainWords& c) {
        constexpr size_t kSmall = (size_t)2 << 20;
        const size_t words = chain_words(n, nrhs) * sizeof(*c.z);
        lead = (lead + 255) / 256 * 256;
        if (words > 0 && !fault_hit(kFaultAlloc)) {
            const bool two = lead + words > kSmall && words <= kSmall;
            if (get(p, two ? lead : lead + words) == MFG_OK) {
                if (two) (void)get(&c.z, chain_words(n, nrhs));
                else c.z = reinterpret_cast<unsigned long long*>(*p + lead);
                return MFG_OK;
            }
        }
        return get(p, lead);
    }
    ~Buffers() {
        for (void* p : ptrs) (void)hipFree(p);
    }
};

int lu_factor_api(int64_t n, float* A, int64_t lda, int32_t* ipiv, int64_t* info, int mode, hipStream_t s) {
    if (n < 0 || lda < std::max<int64_t>(1, n) || (n > 0 && (!A || !ipiv)) || !factor_mode_ok(mode))
        return MFG_ERR_INVALID_ARG;
    if (n > INT32_MAX) return MFG_ERR_UNSUPPORTED;
    if (info) *info = 0;
    if (n == 0) return MFG_OK;
    Buffers buf;
    int32_t* dinfo = nullptr;
    char* scratch = nullptr;
    int st = buf.get(&dinfo, 1);
    if (st == MFG_OK) st = buf.get(&scratch, lu_scratch_bytes(n));
    if (st == MFG_OK) st = lu_factor_impl(n, A, lda, ipiv, dinfo, scratch, mode, s);
    if (st != MFG_OK) return st;
    int32_t h = 0;
    MFG_HIP_CHECK(hipMemcpyAsync(&h, dinfo, sizeof(h), hipMemcpyDeviceToHost, s));
    MFG_HIP_CHECK(hipStreamSynchronize(s));  // before dinfo is freed
    if (info) *info = h;
    return MFG_OK;
}

int lu_solve_api(int64_t n, int64_t nrhs, const float* LU, int64_t ldlu, const int32_t* ipiv, float* B, int64_t ldb,
                 hipStream_t s) {
    if (n < 0 || nrhs < 0 || ldlu < std::max<int64_t>(1, n) || ldb < std::max<int64_t>(1, nrhs) ||
        (n > 0 && (!LU || !ipiv)) || (n > 0 && nrhs > 0 && !B))
        return MFG_ERR_INVALID_ARG;
    if (nrhs > INT32_MAX) return MFG_ERR_UNSUPPORTED;
    if (n == 0 || nrhs == 0) return MFG_OK;
    std::vector<int32_t> perm;
    int st = permutation(n, ipiv, perm, s);
    if (st != MFG_OK) return st;
    Buffers buf;
    char* base = nullptr;
    ChainWords chain;
    if ((st = buf.get_with_chain(&base, (size_t)(n * nrhs + n) * 4, n, nrhs, chain)) != MFG_OK) return st;
    float* tmp = reinterpret_cast<float*>(base);
    int32_t* dperm = reinterpret_cast<int32_t*>(tmp + n * nrhs);
    MFG_HIP_CHECK(hipMemcpyAsync(dperm, perm.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, s));
    if ((st = lu_solve_impl(n, nrhs, LU, ldlu, dperm, B, ldb, tmp, nrhs, chain, s)) != MFG_OK) return st;
    MFG_HIP_CHECK(hipMemcpy2DAsync(B, (size_t)ldb * 4, tmp, (size_t)nrhs * 4, (size_t)nrhs * 4, (size_t)n,
                                   hipMemcpyDeviceToDevice, s));
    MFG_HIP_CHECK(hipStreamSynchronize(s));  // before the buffers are freed
    return MFG_OK;
}

int solve_ir_api(int64_t n, int64_t nrhs, const double* A, int64_t lda, const double* B, int64_t ldb, double* X,
                 int64_t ldx, int mode, int max_iter, double tol, int* iters, double* berr, int64_t* info,
                 hipStream_t s) {
    if (n < 0 || nrhs < 0 || lda < std::max<int64_t>(1, n) || ldb < std::max<int64_t>(1, nrhs) ||
        ldx < std::max<int64_t>(1, nrhs) || (n > 0 && !A) || (n > 0 && nrhs > 0 && (!B || !X)) ||
        !factor_mode_ok(mode) || max_iter < 0 || !(tol >= 0.0))
        return MFG_ERR_INVALID_ARG;
    if (n > INT32_MAX || nrhs > INT32_MAX) return MFG_ERR_UNSUPPORTED;
    if (iters) *iters = 0;
    if (berr) *berr = 0.0;
    if (info) *info = 0;
    if (n == 0 || nrhs == 0) return MFG_OK;
    Buffers buf;
    float *A32 = nullptr, *v = nullptr, *d = nullptr;
    char* scratch = nullptr;
    double *R = nullptr, *rows = nullptr, *nrm = nullptr;
    int32_t *ipiv = nullptr, *dperm = nullptr, *dinfo = nullptr;
    char* base = nullptr;
    ChainWords chain;
    int st;
    if ((st = buf.get(&A32, (size_t)(n * n))) != MFG_OK || (st = buf.get(&v, (size_t)(n * nrhs))) != MFG_OK ||
        (st = buf.get_with_chain(&base, (size_t)(n * nrhs) * 4, n, nrhs, chain)) != MFG_OK ||
        (st = buf.get(&R, (size_t)(n * nrhs))) != MFG_OK ||
        (st = buf.get(&rows, (size_t)n)) != MFG_OK || (st = buf.get(&nrm, (size_t)(3 * nrhs + 1))) != MFG_OK ||
        (st = buf.get(&ipiv, (size_t)n)) != MFG_OK || (st = buf.get(&dperm, (size_t)n)) != MFG_OK ||
        (st = buf.get(&dinfo, 1)) != MFG_OK || (st = buf.get(&scratch, lu_scratch_bytes(n))) != MFG_OK)
        return st;
    d = reinterpret_cast<float*>(base);
    // the factorisation of the FP32 copy, in the given mode
    hipLaunchKernelGGL(f64_to_f32, dim3(blocks(n * n, 256)), dim3(256), 0, s, n, n, A, lda, A32, n);
    MFG_LAUNCH_CHECK();
    if ((st = lu_factor_impl(n, A32, n, ipiv, dinfo, scratch, mode, s)) != MFG_OK) return st;
    int32_t hinfo = 0;
    MFG_HIP_CHECK(hipMemcpyAsync(&hinfo, dinfo, sizeof(hinfo), hipMemcpyDeviceToHost, s));
    std::vector<int32_t> perm;
    if ((st = permutation(n, ipiv, perm, s)) != MFG_OK) return st;  // synchronises
    if (info) *info = hinfo;
    if (hinfo != 0) {
        MFG_HIP_CHECK(hipStreamSynchronize(s));
        return MFG_OK;  // exactly singular factor: no solve (info says where)
    }
    MFG_HIP_CHECK(hipMemcpyAsync(dperm, perm.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, s));
    // |A|_inf and |b_j|_inf, once
    hipLaunchKernelGGL(abs_row_sums, dim3(blocks(n, 4)), dim3(256), 0, s, n, A, lda, rows);
    MFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(col_abs_max, dim3(1), dim3(256), 0, s, n, (int64_t)1, rows, (int64_t)1, nrm + 3 * nrhs);
    MFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(col_abs_max, dim3((unsigned)nrhs), dim3(256), 0, s, n, nrhs, B, ldb, nrm + nrhs);
    MFG_LAUNCH_CHECK();
    // x0 from the factors
    hipLaunchKernelGGL(f64_to_f32, dim3(blocks(n * nrhs, 256)), dim3(256), 0, s, n, nrhs, B, ldb, v, nrhs);
    MFG_LAUNCH_CHECK();
    if ((st = lu_solve_impl(n, nrhs, A32, n, dperm, v, nrhs, d, nrhs, chain, s)) != MFG_OK) return st;
    hipLaunchKernelGGL(accumulate_f64, dim3(blocks(n * nrhs, 256)), dim3(256), 0, s, n, nrhs, d, nrhs, X, ldx, 1);
    MFG_LAUNCH_CHECK();
    std::vector<double> h((size_t)(3 * nrhs + 1));
    double be = INFINITY;
    int it = 0;
    for (;; ++it) {
        // r = b - A x (FP64) and the backward error of x
        hipLaunchKernelGGL(residual_f64, dim3(blocks(n * nrhs, 4)), dim3(256), 0, s, n, nrhs, A, lda, X, ldx, B, ldb,
                           R, nrhs);
        MFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(col_abs_max, dim3((unsigned)nrhs), dim3(256), 0, s, n, nrhs, R, nrhs, nrm);
        MFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(col_abs_max, dim3((unsigned)nrhs), dim3(256), 0, s, n, nrhs, X, ldx, nrm + 2 * nrhs);
        MFG_LAUNCH_CHECK();
        MFG_HIP_CHECK(hipMemcpyAsync(h.data(), nrm, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s));
        MFG_HIP_CHECK(hipStreamSynchronize(s));
        be = 0.0;
        const double anorm = h[(size_t)(3 * nrhs)];
        for (int64_t q = 0; q < nrhs; ++q) {
            const double den = anorm * h[(size_t)(2 * nrhs + q)] + h[(size_t)(nrhs + q)];
            const double e = den > 0.0 ? h[(size_t)q] / den : (h[(size_t)q] > 0.0 ? INFINITY : 0.0);
            be = std::max(be, e);
        }
        if (!(be > tol) || it >= max_iter) break;
        // correction: d = (LU)^-1 P r in FP32, x += d in FP64
        hipLaunchKernelGGL(f64_to_f32, dim3(blocks(n * nrhs, 256)), dim3(256), 0, s, n, nrhs, R, nrhs, v, nrhs);
        MFG_LAUNCH_CHECK();
        if ((st = lu_solve_impl(n, nrhs, A32, n, dperm, v, nrhs, d, nrhs, chain, s)) != MFG_OK) return st;
        hipLaunchKernelGGL(accumulate_f64, dim3(blocks(n * nrhs, 256)), dim3(256), 0, s, n, nrhs, d, nrhs, X, ldx, 0);
        MFG_LAUNCH_CHECK();
    }
    if (iters) *iters = it;
    if (berr) *berr = be;
    return MFG_OK;
}

}  // namespace

#define MFG_SOLVE_GUARD(expr)                \
    try {                                    \
        return (expr);                       \
    } catch (const std::bad_alloc&) {        \
        return MFG_ERR_NO_MEMORY;            \
    } catch (...) {                          \
        return MFG_ERR_INTERNAL;             \
    }

extern "C" int mfg_lu_factor(int64_t n, float* A, int64_t lda, int32_t* ipiv, int64_t* info, int mode,
                             void* stream) {
    MFG_SOLVE_GUARD(lu_factor_api(n, A, lda, ipiv, info, mode, (hipStream_t)stream));
}

extern "C" int mfg_lu_solve(int64_t n, int64_t nrhs, const float* LU, int64_t ldlu, const int32_t* ipiv, float* B,
                            int64_t ldb, void* stream) {
    MFG_SOLVE_GUARD(lu_solve_api(n, nrhs, LU, ldlu, ipiv, B, ldb, (hipStream_t)stream));
}

extern "C" int mfg_solve_ir(int64_t n, int64_t nrhs, const double* A, int64_t lda, const double* B, int64_t ldb,
                            double* X, int64_t ldx, int mode, int max_iter, double tol, int* iters, double* berr,
                            int64_t* info, void* stream) {
    MFG_SOLVE_GUARD(solve_ir_api(n, nrhs, A, lda, B, ldb, X, ldx, mode, max_iter, tol, iters, berr, info,
                                 (hipStream_t)stream));
}
