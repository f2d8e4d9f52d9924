// ring16.h -- the 16-bit GEMM kernel for small output tiles and ragged
// sizes: any M, N, K with 16-byte aligned operand rows.
//
// Same arithmetic as tile16.h (same MFMA, same K order, same epilogue, zeros
// beyond K), so results are bitwise those of every other configuration.
// What bounds it: at these sizes the latency of a stage's loads and the bytes
// each CU draws from L2 (16 KB per 64 x 64 x 64 stage against 128 MFMA
// cycles per SIMD), not the matrix cores.  Hence small tiles, so that many
// CUs draw at once, and several stages or workgroups in flight per CU.
// Measured against the register-staged 64 x 64 tiled kernel it replaced:
// F16 512^3 8.8 -> 4.9 us, 1000^3 15.8 -> 7.8 us, 128 x 128 x 4096
// 48 -> 17 us (0.27 us per stage); SPLIT3 1000^3 41.7 -> 12.9 us.
//   - K moves through a ring of S LDS stages of 64 (each its own __shared__
//     array, so the compiler sees that a read of one stage does not touch the
//     loads still in flight into the others), filled by loads that write LDS
//     directly.  Loads run S-1 stages ahead with one barrier per stage: a
//     short K is in flight as a whole before the first MFMA.
//   - Ragged edges cost no branches in the loop.  Rows past M are clamped
//     (their outputs are not stored).  A's 16-byte pieces and B's rows at or
//     past K are loaded from 16 zero bytes instead, so the last stage is
//     zero-filled.  Where K % 8 != 0 the piece that straddles K is loaded
//     whole (its tail lies in the row's ld extent, in the same aligned 16
//     bytes) and its elements past K are cleared in LDS once the last stage
//     has landed.  B's columns past N reach only outputs that are not stored.
#pragma once

#include <type_traits>

#include "pipe16.h"

namespace mfg {

// Swizzle of 16-byte chunks of a B row of BN halfs: chunk c of row k is kept
// at c ^ F[k % 4].  The transposing read takes, per 16 lanes, 32 bytes of
// each of four consecutive rows; these place the four in different banks.
template <int BN>
__device__ __forceinline__ int ring_swz_b(int k) {
    if constexpr (BN == 64) return (k & 3) * 2;  // F = {0, 2, 4, 6}: rows of 8
    else return swzB(k);
}

// The lane's offset (halfs) in a B plane of its part of the MFMA operand with
// columns nb .. nb + 31 of K rows 0 .. 15 (as read_b_tr; rows 16 ch on are
// 16 ch BN further, rows + 4 at 4 BN).
template <int BN>
__device__ __forceinline__ int ring_offset_b(int nb, int lane) {
    const int w = lane & 15, j = w >> 2, q = w & 3;
    const int n = nb + ((lane >> 4) & 1) * 16 + q * 4;
    const int k1 = (lane >> 5) * 8 + j;  // k1 and k1 + 4 share k % 4
    return k1 * BN + (((n >> 3) ^ ring_swz_b<BN>(k1)) << 3) + (n & 7);
}

template <int BN>
__device__ __forceinline__ u32x4 ring_read_b(const uint16_t* p) {
    i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p);
    i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p + 4 * BN));
    u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
    return u32x4{a[0], a[1], b[0], b[1]};
}

// Keeps a computed offset as one value.  An LDS address then stays array +
// offset + constant; folded into longer chains, the compiler no longer knew
// which array a read touches and waited for every load in flight first.
__device__ __forceinline__ void opaque(int& x) { asm("" : "+v"(x)); }

template <int KIND, int BM, int BN, int WM, int WN, int S>
struct RingCfg {
    static constexpr int BK = 64;
    static constexpr int NW = WM * WN, NT = 64 * NW;
    static constexpr int TMW = BM / WM, TNW = BN / WN;
    static constexpr int FM = TMW / 32, FN = TNW / 32;
    static constexpr int NPA = KT<KIND>::NPA, NPB = KT<KIND>::NPB;
    static constexpr int A_PLANE = BM * BK, B_PLANE = BK * BN;  // halfs
    static constexpr int STAGE = NPA * A_PLANE + NPB * B_PLANE;
    static constexpr int A_INSTR = A_PLANE / 512 / NW, B_INSTR = B_PLANE / 512 / NW;  // 1 KB loads per wave per plane
    static constexpr int LOADS = NPA * A_INSTR + NPB * B_INSTR;
    static constexpr int B_ROWS_PER_INSTR = 512 / BN, B_CPR = BN / 8;
    static_assert(A_PLANE % (512 * NW) == 0 && B_PLANE % (512 * NW) == 0, "tile must split into 1 KB loads");
    static_assert(BN == 64 || BN == 128, "B rows of 128 or 256 bytes");
    static_assert(S == 2 || S == 3, "2 or 3 stages");
    static_assert(S * STAGE * 2 <= 160 * 1024, "LDS budget");
    static_assert(LOADS * (S - 1) <= 63, "vmcnt range");
};

// Global -> LDS loads of 64-deep stages with the edge rules above.  Per-lane
// offsets from the tile's corner (A row m0, B column n0) are fixed for the K
// loop; a stage adds its K offset to the base in scalar registers.
template <class G, int BN>
struct RingLoader {
    const char* a[2];
    const char* b[2];
    int64_t K, ldb2;
    const char* zeros;
    int wid;
    uint32_t offa[G::A_INSTR], offb[G::B_INSTR];
    int ka[G::A_INSTR], kb[G::B_INSTR];  // first K column of the lane's A piece, K row of its B piece, within a stage

    __device__ __forceinline__ void init(const uint16_t* const (&Ap)[2], const uint16_t* const (&Bp)[2], int64_t lda,
                                         int64_t ldb, int64_t M, int64_t N, int64_t K_, int64_t m0, int64_t n0,
                                         int wid_, int lane) {
        wid = __builtin_amdgcn_readfirstlane(wid_);
        K = uniform64(K_);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            a[q] = (const char*)uniform64((int64_t)(Ap[q] ? Ap[q] + m0 * lda : nullptr));
            b[q] = (const char*)uniform64((int64_t)(Bp[q] ? Bp[q] + n0 : nullptr));
        }
        ldb2 = uniform64(ldb * 2);
        zeros = (const char*)kZeros16;
        const int64_t n8 = (N + 7) / 8 * 8;  // <= ldb (a multiple of 8)
#pragma unroll
        for (int i = 0; i < G::A_INSTR; ++i) {
            const int row = (wid * G::A_INSTR + i) * 8 + (lane >> 3);
            const int64_t gm = m0 + row < M ? m0 + row : M - 1;
            ka[i] = ((lane & 7) ^ swz<8>(row)) * 8;
            offa[i] = (uint32_t)(((gm - m0) * lda + ka[i]) * 2);
        }
#pragma unroll
        for (int i = 0; i < G::B_INSTR; ++i) {
            kb[i] = (wid * G::B_INSTR + i) * G::B_ROWS_PER_INSTR + lane / G::B_CPR;
            const int64_t gn = n0 + ((lane % G::B_CPR) ^ ring_swz_b<BN>(kb[i])) * 8;
            offb[i] = (uint32_t)((kb[i] * ldb + (gn < n8 ? gn : n8 - 8) - n0) * 2);
        }
    }

    // The stage starting at k0 (k0 >= K: zeros) into `st`.  Pieces at or past
    // K come from `zeros` instead of the operand.
    __device__ __forceinline__ void load(int64_t k0, uint16_t* st) const {
        const int64_t left = uniform64(K - k0);  // K columns / rows from k0 on
        const int kl = left < 64 ? (int)left : 64;
        const int64_t ka2 = uniform64(k0 * 2), kb2 = uniform64(k0 * ldb2);
#pragma unroll
        for (int q = 0; q < G::NPA; ++q)
#pragma unroll
            for (int i = 0; i < G::A_INSTR; ++i)
                __builtin_amdgcn_global_load_lds((const void*)(ka[i] < kl ? a[q] + ka2 + offa[i] : zeros),
                                                 (lds_void*)(st + q * G::A_PLANE + (wid * G::A_INSTR + i) * 512), 16,
                                                 0, 0);
#pragma unroll
        for (int q = 0; q < G::NPB; ++q)
#pragma unroll
            for (int i = 0; i < G::B_INSTR; ++i)
                __builtin_amdgcn_global_load_lds(
                    (const void*)(kb[i] < kl ? b[q] + kb2 + offb[i] : zeros),
                    (lds_void*)(st + G::NPA * G::A_PLANE + q * G::B_PLANE + (wid * G::B_INSTR + i) * 512), 16, 0, 0);
    }
};

template <int KIND, int BM, int BN, int WM, int WN, int S, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm16_ring(Gemm16Args p, int tiles_m, int tiles_n, int group_m) {
    using T = KT<KIND>;
    using G = RingCfg<KIND, BM, BN, WM, WN, S>;
    constexpr int FM = G::FM, FN = G::FN;
    __shared__ __attribute__((aligned(16))) uint16_t st0[G::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t st1[G::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t st2[S > 2 ? G::STAGE : 8];

    int tm, tn;
    raster(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, group_m, tm, tn);
    const int64_t bz = blockIdx.y;
    const uint16_t* Ap[2];
    const uint16_t* Bp[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        Ap[q] = (q < T::NPA) ? p.A[q] + bz * p.sA : nullptr;
        Bp[q] = (q < T::NPB) ? p.B[q] + bz * p.sB : nullptr;
    }
    float* C = p.C + bz * p.sC;
    const int64_t M = p.M, N = p.N, K = p.K;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN;
    const int64_t KTN = uniform64((K + 63) / 64);
    auto stage = [&](int s) -> uint16_t* { return s == 0 ? st0 : (S == 2 || s == 1) ? st1 : st2; };

    f32x16 hi[FM][FN], lo[FM][FN], rr[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            hi[i][j] = f32x16{};
            if constexpr (T::LO) lo[i][j] = f32x16{};
            if constexpr (T::RR) rr[i][j] = f32x16{};
        }

    RingLoader<G, BN> ld;
    ld.init(Ap, Bp, p.lda, p.ldb, M, N, K, m0, n0, wid, lane);
#pragma unroll
    for (int s = 0; s < S - 1; ++s) ld.load(s * 64, stage(s));

    int oa[FM][4], ob[FN];  // this lane's fragment offsets in a stage's A and B planes
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
        const int row = wm * G::TMW + fm * 32 + (lane & 31);
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            oa[fm][ch] = row * 64 + (((ch * 2 + (lane >> 5)) ^ swz<8>(row)) * 8);
            opaque(oa[fm][ch]);
        }
    }
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        ob[fn] = ring_offset_b<BN>(wn * G::TNW + fn * 32, lane);
        opaque(ob[fn]);
    }

    auto multiply = [&](const uint16_t* st) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            u32x4 a[FM][2], b[FN][2];
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    a[fm][q] = (q < T::NPA) ? *reinterpret_cast<const u32x4*>(st + oa[fm][ch] + q * G::A_PLANE) : zero4();
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    b[fn][q] = (q < T::NPB) ? ring_read_b<BN>(st + ob[fn] + (G::NPA * G::A_PLANE + q * G::B_PLANE + ch * 16 * BN))
                                            : zero4();
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int fn = 0; fn < FN; ++fn) mma_step<KIND>(a[fm], b[fn], hi[fm][fn], lo[fm][fn], rr[fm][fn]);
        }
    };
    // Stage t (slot u), not the last one: wait for this wave's loads of it and
    // its reads of the stage before, barrier (everyone's loads landed;
    // everyone is done with slot u - 1), refill that slot with stage
    // t + S - 1, multiply.
    auto step = [&](auto ucst, int64_t t) {
        constexpr int u = decltype(ucst)::value;
        wait_vmcnt<G::LOADS * (S - 2)>();
        wait_lgkm0();
        bare_barrier();
        ld.load((t + S - 1) * 64, stage((u + S - 1) % S));
        __builtin_amdgcn_sched_barrier(0);  // the loads go out before the MFMAs, not after them
        multiply(stage(u));
    };
    const int64_t last = KTN - 1, whole = last - last % S;
    for (int64_t t = 0; t < whole; t += S) {
        step(std::integral_constant<int, 0>{}, t);
        step(std::integral_constant<int, 1>{}, t + 1);
        if constexpr (S > 2) step(std::integral_constant<int, 2>{}, t + 2);
    }
    if (whole < last) step(std::integral_constant<int, 0>{}, whole);
    if constexpr (S > 2)
        if (whole + 1 < last) step(std::integral_constant<int, 1>{}, whole + 1);

    // the last stage: nothing left to load, and the piece that straddles K to
    // clear (here and not in the loop: a divergent branch there made the
    // compiler wait for every load in flight, in every stage)
    uint16_t* tail = stage((int)(last - whole));
    wait_vmcnt<0>();
    wait_lgkm0();
    bare_barrier();
    if ((K & 7) != 0) {
        clear_straddle<G, BM>(tail, (int)(K - last * 64), tid);
        wait_lgkm0();
        bare_barrier();
    }
    multiply(tail);

    store_tile<FM, FN>(C, p.ldc, M, N, m0 + wm * G::TMW, n0 + wn * G::TNW, lane, p.alpha, p.beta,
                       [&](int fm, int fn, int i) { return combine_at<KIND>(hi[fm][fn], lo[fm][fn], rr[fm][fn], i); });
}

}  // namespace mfg
