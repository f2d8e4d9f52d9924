// gemm_f32.hip -- single-precision GEMM on the gfx950 matrix cores
// (v_mfma_f32_32x32x2_f32): the FP32 comparator of the half-precision modes
// (the paper's single-precision GEMM, Sec. VII.A and the error reference of
// Sec. VI).
//
// Accumulation order of an output element, shared by every kernel here: K
// is walked in blocks of 8; inside a block, four MFMAs j = 0..3 each add the
// products at k = kb + j (lane half 0) and k = kb + 4 + j (lane half 1).
#include "internal.h"
#include "pipe16.h"
#include "ring16.h"
#include "runtime.h"

namespace mfg {

__device__ __forceinline__ f32x4 load_row4(const float* p, bool valid, int64_t off, int64_t remaining,
                                           bool vec) {
    if (!valid || remaining <= 0) return f32x4{0.f, 0.f, 0.f, 0.f};
    if (vec && remaining >= 4) return *reinterpret_cast<const f32x4*>(p + off);
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (j < remaining) ? p[off + j] : 0.0f;
    return v;
}

// One wavefront per 32x32 tile, operands from global memory.
__global__ __launch_bounds__(64) void gemmf32_simple(GemmF32Args p, int vecA) {
    const int lane = threadIdx.x;
    const int r = lane & 31, g = lane >> 5;
    const int64_t bz = blockIdx.z;
    const int64_t m0 = (int64_t)blockIdx.y * 32, n0 = (int64_t)blockIdx.x * 32;
    const float* A = p.A + bz * p.sA;
    const float* B = p.B + bz * p.sB;
    float* C = p.C + bz * p.sC;
    const int64_t am = m0 + r, bn = n0 + r;
    f32x16 acc = {};
    for (int64_t kb = 0; kb < p.K; kb += 8) {
        const int64_t k = kb + g * 4;
        f32x4 a = load_row4(A, am < p.M, am * p.lda + k, p.K - k, vecA != 0);
        f32x4 b;
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = (bn < p.N && k + j < p.K) ? B[(k + j) * p.ldb + bn] : 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = mma_32x32x2_f32(a[j], b[j], acc);
    }
    store_blocks<1>(C, p.ldc, p.M, p.N, m0, n0, lane, p.alpha, p.beta, [&](int, int i) { return acc[i]; });
}

__device__ __forceinline__ int xcd_remap_f32(int bid, int nblk) {
    const int per = nblk / 8, rem = nblk % 8;
    const int xcd = bid % 8, idx = bid / 8;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// Tiled FP32 kernel: BM x BN tile, BK = 32 (eight 16-byte chunks per LDS
// row, XOR-swizzled), 2x2 wavefronts, LDS double buffer.  B is transposed
// through registers into B^T [BN][BK] (4 rows x 4 columns per thread).
template <int BM, int BN>
__global__ __launch_bounds__(256) void gemmf32_tiled(GemmF32Args p, int tiles_m, int tiles_n, int group_m) {
    constexpr int BK = 32, CPR = 8, NT = 256, WM = 2, WN = 2;
    constexpr int TMW = BM / WM, TNW = BN / WN, FM = TMW / 32, FN = TNW / 32;
    constexpr int A_PER_T = BM * CPR / NT;
    constexpr int B_UNITS = (BK / 4) * (BN / 4);
    constexpr int B_PER_T = B_UNITS / NT;
    constexpr int STAGE = (BM + BN) * BK;
    static_assert(B_UNITS % NT == 0 && (BM * CPR) % NT == 0, "tile/thread split");
    extern __shared__ __attribute__((aligned(16))) float ldsf[];

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN;
    int tm, tn;
    {
        const int lid = xcd_remap_f32(blockIdx.x, gridDim.x);
        const int group = group_m * tiles_n, gid = lid / group, first_m = gid * group_m;
        const int gm = min(tiles_m - first_m, group_m), in = lid - gid * group;
        tm = first_m + in % gm;
        tn = in / gm;
    }
    const int64_t bz = blockIdx.y;
    const float* A = p.A + bz * p.sA;
    const float* B = p.B + bz * p.sB;
    float* C = p.C + bz * p.sC;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int64_t M = p.M, N = p.N, K = p.K;
    const bool mn_interior = (m0 + BM <= M) && (n0 + BN <= N);

    f32x4 ra[A_PER_T];
    f32x4 rb[B_PER_T][4];
    auto gload = [&](int64_t k0) {
        const bool interior = mn_interior && (k0 + BK <= K);
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) {
            const int id = tid + i * NT, row = id / CPR, c = id % CPR;
            const int64_t gm = m0 + row, gk = k0 + c * 4;
            ra[i] = interior ? *reinterpret_cast<const f32x4*>(A + gm * p.lda + gk)
                             : load_row4(A, gm < M, gm * p.lda + gk, K - gk, true);
        }
#pragma unroll
        for (int u = 0; u < B_PER_T; ++u) {
            const int uid = tid + u * NT;
            const int qn = uid % (BN / 4), gk_ = uid / (BN / 4);
            const int64_t gn = n0 + qn * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t gk = k0 + gk_ * 4 + i;
                rb[u][i] = interior ? *reinterpret_cast<const f32x4*>(B + gk * p.ldb + gn)
                                    : load_row4(B, gk < K, gk * p.ldb + gn, N - gn, true);
            }
        }
    };
    auto swrite = [&](int stage) {
        float* As = ldsf + stage * STAGE;
        float* Bs = As + BM * BK;
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) {
            const int id = tid + i * NT, row = id / CPR, c = id % CPR;
            *reinterpret_cast<f32x4*>(As + row * BK + ((c ^ swz<CPR>(row)) * 4)) = ra[i];
        }
#pragma unroll
        for (int u = 0; u < B_PER_T; ++u) {
            const int uid = tid + u * NT;
            const int qn = uid % (BN / 4), gk_ = uid / (BN / 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = qn * 4 + j;
                f32x4 v = {rb[u][0][j], rb[u][1][j], rb[u][2][j], rb[u][3][j]};
                *reinterpret_cast<f32x4*>(Bs + n * BK + ((gk_ ^ swz<CPR>(n)) * 4)) = v;
            }
        }
    };

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};

    auto compute = [&](int stage) {
        const float* As = ldsf + stage * STAGE;
        const float* Bs = As + BM * BK;
#pragma unroll
        for (int kk = 0; kk < BK / 8; ++kk) {
            const int c = kk * 2 + (lane >> 5);
            f32x4 af[FM], bf[FN];
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                const int row = wm * TMW + fm * 32 + (lane & 31);
                af[fm] = *reinterpret_cast<const f32x4*>(As + row * BK + ((c ^ swz<CPR>(row)) * 4));
            }
#pragma unroll
            for (int fn = 0; fn < FN; ++fn) {
                const int n = wn * TNW + fn * 32 + (lane & 31);
                bf[fn] = *reinterpret_cast<const f32x4*>(Bs + n * BK + ((c ^ swz<CPR>(n)) * 4));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mma_32x32x2_f32(af[fm][j], bf[fn][j], acc[fm][fn]);
        }
    };

    const int64_t KTN = cdiv(K, BK);
    if (KTN > 0) {
        gload(0);
        swrite(0);
        __syncthreads();
        for (int64_t kt = 0; kt < KTN; ++kt) {
            const int cur = (int)(kt & 1);
            if (kt + 1 < KTN) gload((kt + 1) * BK);
            compute(cur);
            if (kt + 1 < KTN) swrite(cur ^ 1);
            __syncthreads();
        }
    }
    store_tile<FM, FN>(C, p.ldc, M, N, m0 + wm * TMW, n0 + wn * TNW, lane, p.alpha, p.beta,
                       [&](int fm, int fn, int i) { return acc[fm][fn][i]; });
}

// ---------------------------------------------------------------------------
// gemmf32_ring: any M, N, K and any row alignment.  Bound by the matrix
// cores: v_mfma_f32_32x32x2 takes 64 cycles, 256 of them per 64 x 64 x 32
// stage against 16 KB of operands, so what matters is that nothing else
// holds the wave between MFMAs.  Both operands go straight into LDS
// (S stages of 32, S-1 ahead, one barrier per stage) in their row-major
// layout: A rows as in gemmf32_tiled; B is read element by element, four
// ds_read_b32 per 32 columns and 8-deep chunk, so it needs no transpose
// through registers.  The two lane halves read B rows k and k + 4: those are
// kept 128 bytes apart modulo 256 (columns ^ 32, for BN = 32 row pairs
// swapped), so the read is free of bank conflicts.
// VEC: 16-byte loads (aligned rows, K % 4 == 0); otherwise 4-byte loads, four
// times as many, which the MFMAs still cover.  K columns of A and rows of B
// at or past K are loaded from zeros, M rows and N columns past the edge are
// clamped to the last one.
// Measured against the register-staged 128 x 128 kernel and, for small or
// unaligned problems, the simple one: 2048^3 157 -> 139 us (124 TFLOP/s),
// 3000^3 764 -> 465, 1000^3 77 -> 25, 256^3 15 -> 7.8, 8192^3 8.68 -> 8.40
// ms, 1772 x 2736 x 1437 with odd ld 435 -> 174.
template <int BM, int BN, int WM, int WN, int S, bool VEC>
struct F32Cfg {
    static constexpr int BK = 32, NW = WM * WN, NT = 64 * NW;
    static constexpr int TMW = BM / WM, TNW = BN / WN, FM = TMW / 32, FN = TNW / 32;
    static constexpr int A_TILE = BM * BK, B_TILE = BK * BN, STAGE = A_TILE + B_TILE;  // floats
    static constexpr int E = VEC ? 4 : 1;  // elements per lane and load
    static constexpr int A_INSTR = A_TILE / (64 * E) / NW, B_INSTR = B_TILE / (64 * E) / NW;
    static constexpr int LOADS = A_INSTR + B_INSTR;
    static_assert(A_TILE % (64 * 4 * NW) == 0 && B_TILE % (64 * 4 * NW) == 0, "tile must split into loads");
    static_assert(BN == 64 || BN == 128, "B rows of 256 or 512 bytes");
    static_assert(S >= 2 && S <= 3 && S * STAGE * 4 <= 160 * 1024, "LDS budget");
    static_assert(LOADS * (S - 1) <= 63, "vmcnt range");
};

// LDS position (floats) of B element (k, n) within a stage's B tile.
template <int BN>
__device__ __forceinline__ int f32_b_at(int k, int n) {
    const int h = (k >> 2) & 1;
    return k * BN + (n ^ (h << 5));
}

template <int BM, int BN, int WM, int WN, int S, bool VEC, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemmf32_ring(GemmF32Args p, int tiles_m, int tiles_n,
                                                                  int group_m) {
    using G = F32Cfg<BM, BN, WM, WN, S, VEC>;
    constexpr int FM = G::FM, FN = G::FN, E = G::E;
    __shared__ __attribute__((aligned(16))) float st0[G::STAGE];
    __shared__ __attribute__((aligned(16))) float st1[G::STAGE];
    __shared__ __attribute__((aligned(16))) float st2[S > 2 ? G::STAGE : 4];
    auto stage = [&](int s) -> float* { return s == 0 ? st0 : (S == 2 || s == 1) ? st1 : st2; };

    int tm, tn;
    raster(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, group_m, tm, tn);
    const int64_t bz = blockIdx.y;
    const int64_t M = p.M, N = p.N, K = uniform64(p.K), lda = p.lda, ldb = p.ldb;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WN, wn = wid % WN, r = lane & 31, g = lane >> 5;

    // per-lane sources: byte offset from the tile's corner and K index within a stage
    const char* a = (const char*)uniform64((int64_t)(p.A + bz * p.sA + m0 * lda));
    const char* b = (const char*)uniform64((int64_t)(p.B + bz * p.sB + n0));
    const int64_t ldb4 = uniform64(ldb * 4);
    int64_t offa[G::A_INSTR], offb[G::B_INSTR];
    int ka[G::A_INSTR], kb[G::B_INSTR];
#pragma unroll
    for (int i = 0; i < G::A_INSTR; ++i) {
        const int at = ((wid * G::A_INSTR + i) * 64 + lane) * E, row = at >> 5, w = at & 31;
        ka[i] = (((w >> 2) ^ swz<8>(row)) << 2) + (w & 3);
        offa[i] = (((m0 + row < M ? m0 + row : M - 1) - m0) * lda + ka[i]) * 4;
    }
    const int64_t nlast = VEC ? (N + 3) / 4 * 4 - 4 : N - 1;  // last load's first column (N up to 4 <= ldb)
#pragma unroll
    for (int i = 0; i < G::B_INSTR; ++i) {
        const int at = ((wid * G::B_INSTR + i) * 64 + lane) * E, row = at / BN, n = at % BN;
        const int h = (row >> 2) & 1;
        kb[i] = row;
        const int64_t gn = n0 + (n ^ (h << 5));
        offb[i] = (kb[i] * ldb + (gn < nlast ? gn : nlast) - n0) * 4;
    }
    auto load_lds = [](const char* src, float* dst) {
        if constexpr (VEC) __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)dst, 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)dst, 4, 0, 0);
    };
    auto load = [&](int64_t k0, float* st) {
        const int kl = (int)min(uniform64(K - k0), (int64_t)G::BK);  // <= 0 past the last stage: zeros
        const int64_t ao = uniform64(k0 * 4), bo = uniform64(k0 * ldb4);
#pragma unroll
        for (int i = 0; i < G::A_INSTR; ++i)
            load_lds(ka[i] < kl ? a + ao + offa[i] : (const char*)kZeros16, st + (wid * G::A_INSTR + i) * 64 * E);
#pragma unroll
        for (int i = 0; i < G::B_INSTR; ++i)
            load_lds(kb[i] < kl ? b + bo + offb[i] : (const char*)kZeros16,
                     st + G::A_TILE + (wid * G::B_INSTR + i) * 64 * E);
    };

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};

    int oa[FM][4], ob[FN][2];  // this lane's fragment offsets in a stage
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int row = wm * G::TMW + fm * 32 + r;
            oa[fm][kk] = row * 32 + (((kk * 2 + g) ^ swz<8>(row)) * 4);
            opaque(oa[fm][kk]);
        }
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int o = 0; o < 2; ++o) {  // rows 4 g + o; + 2 at 2 BN, + 8 kk at 8 BN kk
            ob[fn][o] = G::A_TILE + f32_b_at<BN>(4 * g + o, wn * G::TNW + fn * 32 + r);
            opaque(ob[fn][o]);
        }
    auto multiply = [&](const float* st) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            f32x4 af[FM];
            float bf[FN][4];
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) af[fm] = *reinterpret_cast<const f32x4*>(st + oa[fm][kk]);
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
                for (int j = 0; j < 4; ++j) bf[fn][j] = st[ob[fn][j & 1] + (kk * 8 + (j & 2)) * BN];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mma_32x32x2_f32(af[fm][j], bf[fn][j], acc[fm][fn]);
        }
    };

#pragma unroll
    for (int s = 0; s < S - 1; ++s) load(s * G::BK, stage(s));
    // stage t (slot u) as in gemm16_ring
    auto step = [&](auto ucst, int64_t t) {
        constexpr int u = decltype(ucst)::value;
        wait_vmcnt<G::LOADS * (S - 2)>();
        wait_lgkm0();
        bare_barrier();
        load((t + S - 1) * G::BK, stage((u + S - 1) % S));
        __builtin_amdgcn_sched_barrier(0);
        multiply(stage(u));
    };
    const int64_t last = uniform64((K + G::BK - 1) / G::BK) - 1, whole = last - last % S;
    for (int64_t t = 0; t < whole; t += S) {
        step(std::integral_constant<int, 0>{}, t);
        step(std::integral_constant<int, 1>{}, t + 1);
        if constexpr (S > 2) step(std::integral_constant<int, 2>{}, t + 2);
    }
    if (whole < last) step(std::integral_constant<int, 0>{}, whole);
    if constexpr (S > 2)
        if (whole + 1 < last) step(std::integral_constant<int, 1>{}, whole + 1);
    wait_vmcnt<0>();
    wait_lgkm0();
    bare_barrier();
    multiply(stage((int)(last - whole)));

    store_tile<FM, FN>(p.C + bz * p.sC, p.ldc, M, N, m0 + wm * G::TMW, n0 + wn * G::TNW, lane, p.alpha, p.beta,
                       [&](int fm, int fn, int i) { return acc[fm][fn][i]; });
}

struct CfgF32 {
    const char* name;
    int bm, bn, group_m;
};
// Index 1 is the ring kernels (tile by pick_ring_f32); 2 the register-staged tile.
static const CfgF32 kCfgF32[] = {
    {"simple32", 0, 0, 0},
    {"rk32g8", 64, 64, 8},
    {"t256x128k32w2x2g8", 256, 128, 8},
};

int num_configs_f32() { return (int)(sizeof(kCfgF32) / sizeof(kCfgF32[0])); }
const char* config_f32_name(int cfg) { return (cfg >= 0 && cfg < num_configs_f32()) ? kCfgF32[cfg].name : nullptr; }

template <int BM, int BN>
static int launch_f32_tiled(const GemmF32Args& a, int64_t batch, int group_m, hipStream_t s) {
    constexpr int lds = 2 * (BM + BN) * 32 * 4;
    auto kern = gemmf32_tiled<BM, BN>;
    static bool attr_set = false;
    if (!attr_set) {
        MFG_HIP_CHECK(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_set = true;
    }
    const int tiles_m = (int)cdiv(a.M, BM), tiles_n = (int)cdiv(a.N, BN);
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n, (unsigned)batch), dim3(256), lds, s, a, tiles_m, tiles_n,
                       group_m);
    MFG_LAUNCH_CHECK();
    return MFG_OK;
}

template <int BM, int BN, int S, bool VEC, int OCC>
static int launch_f32_ring(const GemmF32Args& a, int64_t batch, int group_m, hipStream_t s) {
    const int tiles_m = (int)cdiv(a.M, BM), tiles_n = (int)cdiv(a.N, BN);
    hipLaunchKernelGGL((gemmf32_ring<BM, BN, 2, 2, S, VEC, OCC>), dim3(tiles_m * tiles_n, (unsigned)batch), dim3(256), 0,
                       s, a, tiles_m, tiles_n, group_m);
    MFG_LAUNCH_CHECK();
    return MFG_OK;
}

bool config_f32_ok(int cfg, int64_t ldc, bool vec_ok) {
    if (cfg < 0 || cfg >= num_configs_f32()) return false;
    return cfg == 0 || (vec_ok && buffer_ldc_ok(ldc));
}

int launch_gemm_f32(int cfg, const GemmF32Args& a, int64_t batch, bool vec_ok, hipStream_t s, bool any_rows) {
    if (fault_hit(kFaultLaunch)) return hip_fail(hipErrorLaunchFailure);  // injected (tests)
    if (cfg < 0 || cfg >= num_configs_f32()) return MFG_ERR_INVALID_ARG;
    if (cfg != 0 && ((!vec_ok && !any_rows) || !buffer_ldc_ok(a.ldc))) return MFG_ERR_UNSUPPORTED;
    const CfgF32& c = kCfgF32[cfg];
    if (cfg == 0) {
        dim3 grid((unsigned)cdiv(a.N, 32), (unsigned)cdiv(a.M, 32), (unsigned)batch);
        hipLaunchKernelGGL(gemmf32_simple, grid, dim3(64), 0, s, a, vec_ok ? 1 : 0);
        MFG_LAUNCH_CHECK();
        return MFG_OK;
    }
    if (cfg == 1) {
        const bool v = vec_ok && a.K % 4 == 0;  // whole 16-byte pieces
        switch (pick_ring_f32(a.M, a.N, a.K, batch, v)) {
            case 2: return v ? launch_f32_ring<128, 128, 2, true, 2>(a, batch, c.group_m, s)
                             : launch_f32_ring<128, 128, 2, false, 2>(a, batch, c.group_m, s);
            case 1: return launch_f32_ring<64, 128, 3, true, 2>(a, batch, c.group_m, s);
            default:
                if (a.K <= 64)  // one or two stages: more workgroups per CU instead of a third stage
                    return v ? launch_f32_ring<64, 64, 2, true, 3>(a, batch, c.group_m, s)
                             : launch_f32_ring<64, 64, 2, false, 3>(a, batch, c.group_m, s);
                return v ? launch_f32_ring<64, 64, 3, true, 2>(a, batch, c.group_m, s)
                         : launch_f32_ring<64, 64, 3, false, 2>(a, batch, c.group_m, s);
        }
    }
    return launch_f32_tiled<256, 128>(a, batch, c.group_m, s);
}

}  // namespace mfg
