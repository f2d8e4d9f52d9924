// capi.cpp -- the exported C ABI of libmfgemm (see include/mfgemm.h):
// validation, operand conversion into the per-stream workspace, tile
// configuration choice and kernel dispatch.  No exception crosses the ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "internal.h"
#include "runtime.h"

namespace mfg {

static bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
static int64_t up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

static int kind_of(int m) {
    switch (m) {
        case MFG_F16: return K_F16;
        case MFG_BF16: return K_BF16;
        case MFG_F16_REFINE_A: return K_REFINE_A;
        case MFG_F16_SPLIT3: return K_SPLIT3;
        case MFG_F16_SPLIT4: return K_SPLIT4;
        case MFG_BF16_SPLIT3: return K_BF16_SPLIT3;
        default: return -1;
    }
}

static bool two_planes_a(int m) {
    return m == MFG_F16_REFINE_A || m == MFG_F16_SPLIT3 || m == MFG_F16_SPLIT4 || m == MFG_BF16_SPLIT3;
}
static bool two_planes_b(int m) { return m == MFG_F16_SPLIT3 || m == MFG_F16_SPLIT4 || m == MFG_BF16_SPLIT3; }
static int npa(int m) { return two_planes_a(m) ? 2 : 1; }
static int npb(int m) { return two_planes_b(m) ? 2 : 1; }

// Write the 16-bit planes of `mode` for an FP32 matrix X (rows x cols).
static int convert16(int m, int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* p0, uint16_t* p1,
                     int64_t ldo, bool split, hipStream_t s) {
    if (m == MFG_BF16) return launch_round_bf16(rows, cols, X, ldx, p0, ldo, s);
    if (split && m == MFG_BF16_SPLIT3) return launch_split_bf16(rows, cols, X, ldx, p0, p1, ldo, nullptr, s);
    if (split) return launch_split_f16(rows, cols, X, ldx, p0, p1, ldo, nullptr, s);
    return launch_round_f16(rows, cols, X, ldx, p0, ldo, s);
}

// ConvJob::kind of an operand of mode m (split: head and residual planes).
static int conv_kind(int m, bool split) { return (split ? 2 : 0) + ((m == MFG_BF16 || m == MFG_BF16_SPLIT3) ? 1 : 0); }

// The planes of A (M x K) and B (K x N) in one launch (a1, b1: null for an
// operand with one plane), K padded with zeros to kp columns of A and rows of
// B (kp == K: none).
static int convert16_pair(int m, int64_t M, int64_t N, int64_t K, int64_t kp, const float* A, int64_t lda,
                          const float* B, int64_t ldb, uint16_t* a0, uint16_t* a1, int64_t ldk, uint16_t* b0,
                          uint16_t* b1, int64_t ldn, hipStream_t s) {
    const ConvJob ja{A, a0, lda, ldk, M, K, M, kp, a1 ? a1 - a0 : 0, conv_kind(m, a1 != nullptr), 0};
    const ConvJob jb{B, b0, ldb, ldn, K, N, kp, N, b1 ? b1 - b0 : 0, conv_kind(m, b1 != nullptr), 0};
    int st = launch_convert_pair(ja, jb, s);
    if (st != MFG_ERR_UNSUPPORTED || kp != K) return st;
    if ((st = convert16(m, M, K, A, lda, a0, a1, ldk, a1 != nullptr, s)) != MFG_OK) return st;
    return convert16(m, K, N, B, ldb, b0, b1, ldn, b1 != nullptr, s);
}

int convert_operands(int m, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, void* wa, int64_t lda_c,
                     const float* B, int64_t ldb, void* wb, int64_t ldb_c, hipStream_t s) {
    if (M > 0 && N > 0 && K > 0 && kind_of(m) >= 0) {
        uint16_t *a0 = static_cast<uint16_t*>(wa), *b0 = static_cast<uint16_t*>(wb);
        return convert16_pair(m, M, N, K, K, A, lda, B, ldb, a0, npa(m) == 2 ? a0 + M * lda_c : nullptr, lda_c, b0,
                              npb(m) == 2 ? b0 + K * ldb_c : nullptr, ldb_c, s);
    }
    if (M > 0 && N > 0 && K > 0 && m == MFG_FP8_E4M3) {
        uint8_t *qa = static_cast<uint8_t*>(wa), *qb = static_cast<uint8_t*>(wb);
        const QuantJob ja{A, qa, reinterpret_cast<float*>(qa + mfg_fp8_scale_offset(M, lda_c)), M, K, lda, lda_c, M, K, 0};
        const QuantJob jb{B, qb, reinterpret_cast<float*>(qb + mfg_fp8_scale_offset(K, ldb_c)), K, N, ldb, ldb_c, K, N, 0};
        return launch_quantize_fp8_pair(ja, &jb, s);
    }
    const int st = mfg_convert(M, K, A, lda, wa, lda_c, m, s);
    return st != MFG_OK ? st : mfg_convert(K, N, B, ldb, wb, ldb_c, m == MFG_F16_REFINE_A ? MFG_F16 : m, s);
}

// gemm_impl's `config`: an index of the mode's menu, the tuned table's entry or
// else the default choice (-1), or the default choice whatever the table holds.
constexpr int kConfigDefault = -2;
static int tuned(int config, int m, int64_t M, int64_t N, int64_t K) {
    return config == kConfigDefault ? -1 : tuned_lookup(m, M, N, K);
}

// The tuned table is keyed by size buckets, so its entry may name a
// configuration that does not serve this particular shape (e.g. K % 64 != 0
// in a bucket tuned on K % 64 == 0): then the default choice is used.
// kp: the K the kernel will run (K, or padded).
static int choose16(int m, int config, int64_t M, int64_t N, int64_t K, int64_t kp, int64_t ldc, bool vec) {
    if (config >= 0) return config;
    const int t = tuned(config, m, M, N, K);
    if (t >= 0 && config16_ok(kind_of(m), t, M, N, K, ldc, vec)) return t;
    return pick_config16(kind_of(m), M, N, kp, vec);
}

// Layout of the 16-bit planes a call converts FP32 operands into: K as the
// kernel will run it, leading dimensions of A's and B's planes.
// Workspace planes of K >= 256 take K padded with zeros to whole 64-deep
// stages (adding zero products changes no bit of an accumulator) and rows
// of whole 128-byte lines, so they run on the kernels for whole stages
// (F16 2048^3: 22.3 us, 24.4 us on the variant for any K).  Below that the
// padding would be over a quarter of the conversion's writes.  Not in the
// fixed array, whose capacity is stated without it, nor beyond the limits
// of one conversion launch and of the tiled kernels.
struct Planes16 {
    int64_t kp, ldk, ldn;
};
static Planes16 planes16(int64_t M, int64_t N, int64_t K, bool fixed) {
    const int64_t k64 = up(K, 64), n64 = N >= 256 ? up(N, 64) : up(N, 8);
    const bool pad = !fixed && K >= 256 && operand_ld_ok(k64, n64) && k64 / 8 * M < ((int64_t)1 << 31) &&
                     cdiv(N, 8) * k64 < ((int64_t)1 << 31);
    if (pad) return {k64, k64, n64};
    return {K, up(K, 8), up(N, 8)};
}

// BF16_SPLIT6 runs the BF16 kernels over K' = 6 * up(K, 64); its tuned
// entries are keyed by its own mode and the caller's K.
static int choose_split6(int config, int64_t M, int64_t N, int64_t K, int64_t ldc, bool vec) {
    if (config >= 0) return config;
    const int64_t kk = 6 * up(K, 64);
    const int t = tuned(config, MFG_BF16_SPLIT6, M, N, K);
    if (t >= 0 && config16_ok(K_BF16, t, M, N, kk, ldc, vec)) return t;
    return pick_config16(K_BF16, M, N, kk, vec);
}

// The storage a call converts its operands into: the per-stream workspace
// (grown with hipMalloc, held by a lease), or caller-provided device memory
// of a fixed capacity (the allocation-free entry point).
struct ExtWs {
    void* ptr;
    size_t cap;
};
struct CallWs {
    std::unique_ptr<WsLease> lease;
    void* ptr = nullptr;
};
static int call_ws(hipStream_t s, size_t bytes, const ExtWs* ext, CallWs& w) {
    if (ext) {
        if (bytes > ext->cap) return MFG_ERR_UNSUPPORTED;
        w.ptr = ext->ptr;
        return MFG_OK;
    }
    w.lease.reset(new WsLease(s, bytes));
    if (!w.lease->ptr()) return w.lease->status();
    w.ptr = w.lease->ptr();
    return MFG_OK;
}

// Whether stream s is being captured.
static bool capturing(hipStream_t s) {
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &c) == hipSuccess) return c != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;  // (the default stream beside another stream's capture)
}

// ran: receives the index of the configuration that was launched.
static int gemm_impl(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                     float* C, int64_t ldc, float alpha, float beta, int mode, int config, hipStream_t s,
                     const ExtWs* ext = nullptr, int* ran = nullptr) {
    int st = validate_gemm(M, N, K, A, lda, B, ldb, C, ldc, mode);
    if (st != MFG_OK) return st;
    const int m = mode & MFG_MODE_MASK;
    const bool pre = (mode & MFG_IN_PRECONVERTED) != 0;
    if (M == 0 || N == 0) return MFG_OK;
    if (K == 0 || alpha == 0.0f) return launch_scale_c(M, N, C, ldc, beta, 1, 0, s);

    if (m == MFG_F32) {
        GemmF32Args a{};
        a.M = M, a.N = N, a.K = K;
        a.A = static_cast<const float*>(A), a.B = static_cast<const float*>(B), a.C = C;
        a.lda = lda, a.ldb = ldb, a.ldc = ldc, a.alpha = alpha, a.beta = beta;
        const bool vec = al16(A) && al16(B) && lda % 4 == 0 && ldb % 4 == 0;
        int cfg = config;
        if (cfg < 0) {
            const int t = tuned(config, m, M, N, K);
            cfg = (t >= 0 && config_f32_ok(t, ldc, vec)) ? t : buffer_ldc_ok(ldc) ? pick_config_f32(M, N, K, vec && K % 4 == 0) : 0;
        }
        if (ran) *ran = cfg;
        return launch_gemm_f32(cfg, a, 1, vec, s, config < 0);
    }

    if (m == MFG_FP8_E4M3) {
        GemmF8Args a{};
        a.M = M, a.N = N, a.K = K, a.C = C, a.ldc = ldc, a.alpha = alpha, a.beta = beta;
        auto choose = [&](bool vec) {
            if (config >= 0) return config;
            const int t = tuned(config, m, M, N, K);
            if (t >= 0 && config_f8_ok(t, M, N, K, ldc, vec)) return t;
            return pick_config_f8(M, N, K, vec, pre);
        };
        const int64_t k128 = up(K, 128), ldt = k128;         // ld of the transposed B codes
        const int64_t bT = up(N * ldt, 256);
        if (pre) {
            a.A = static_cast<const uint8_t*>(A), a.lda = lda;
            a.B = static_cast<const uint8_t*>(B), a.ldb = ldb;
            a.sa = reinterpret_cast<const float*>(a.A + mfg_fp8_scale_offset(M, lda));
            a.sb = reinterpret_cast<const float*>(a.B + mfg_fp8_scale_offset(K, ldb));
            const bool vec = al16(A) && lda % 16 == 0 && buffer_ldc_ok(ldc) && lda < kF8LdLimit && ldt < kF8LdLimit;
            int cfg = choose(vec);
            if (cfg < 0 || cfg >= num_configs_f8()) return MFG_ERR_INVALID_ARG;
            if (f8_config_needs_bt(cfg) && (!vec || (config >= 0 && K % 128 != 0))) return MFG_ERR_UNSUPPORTED;
            // Ragged K and grids under 64 tiles of 128 x 128 are served whatever the
            // storage and the size: by the simple kernel, which reads B's codes as
            // they are, where Bt would exceed the fixed array or the transpose's grid
            // or there is no memory for it, and under capture (a graph would hold the
            // workspace's address past its next growth)
            const bool bare = config < 0 && (K % 128 != 0 || cdiv(M, 128) * cdiv(N, 128) < 64);
            if (bare && ((ext && (size_t)bT > ext->cap) || k128 / 64 > 65535 || (!ext && capturing(s)))) cfg = 0;
            if (ran) *ran = cfg;
            if (!f8_config_needs_bt(cfg)) return launch_gemm_f8(cfg, a, vec, s);
            CallWs ws;
            st = call_ws(s, (size_t)bT, ext, ws);
            if (st == MFG_ERR_NO_MEMORY && bare) {
                if (ran) *ran = 0;
                return launch_gemm_f8(0, a, vec, s);
            }
            if (st != MFG_OK) return st;
            uint8_t* bt = static_cast<uint8_t*>(ws.ptr);
            if ((st = launch_transpose_b8(K, k128, N, a.B, ldb, bt, ldt, s)) != MFG_OK) return st;
            a.Bt = bt, a.ldbt = ldt;
            return launch_gemm_f8(cfg, a, vec, s, config < 0);
        }
        // Workspace codes: A with rows of whole 128-deep stages, zero-filled, and
        // B quantised straight into the K-contiguous layout likewise (zero codes
        // add nothing), so every size runs on the tiled kernels.  Explicit and
        // tuned configurations are judged on the caller's K.
        const float *Af = static_cast<const float*>(A), *Bf = static_cast<const float*>(B);
        const bool vec8 = buffer_ldc_ok(ldc) && k128 < kF8LdLimit;
        int cfg = choose(vec8);
        if (cfg < 0 || cfg >= num_configs_f8()) return MFG_ERR_INVALID_ARG;
        if (f8_config_needs_bt(cfg) && config >= 0 && K % 128 != 0) return MFG_ERR_UNSUPPORTED;
        const int64_t bA = mfg_fp8_scale_offset(M, k128) + 4 * cdiv(M, MFG_FP8_TILE) * cdiv(K, MFG_FP8_TILE);
        const int64_t bS = 4 * cdiv(K, MFG_FP8_TILE) * cdiv(N, MFG_FP8_TILE);
        const size_t tiled_bytes = (size_t)(up(bA, 256) + up(bS, 256) + bT);
        // the fixed array's capacity is stated for unpadded codes: a call whose
        // padding would not fit runs on the simple kernel
        if (config < 0 && ext && tiled_bytes > ext->cap && (K % 128 != 0 || cfg == 2)) cfg = 0;
        if (ran) *ran = cfg;
        if (f8_config_needs_bt(cfg)) {
            CallWs ws;
            if ((st = call_ws(s, tiled_bytes, ext, ws)) != MFG_OK) return st;
            uint8_t* qa = static_cast<uint8_t*>(ws.ptr);
            float* sa = reinterpret_cast<float*>(qa + mfg_fp8_scale_offset(M, k128));
            float* sb = reinterpret_cast<float*>(qa + up(bA, 256));
            uint8_t* bt = qa + up(bA, 256) + up(bS, 256);
            const QuantJob ja{Af, qa, sa, M, K, lda, k128, M, k128, 0}, jb{Bf, bt, sb, K, N, ldb, ldt, k128, N, 1};
            if ((st = launch_quantize_fp8_pair(ja, &jb, s)) != MFG_OK) return st;
            a.K = k128;
            a.A = qa, a.lda = k128, a.sa = sa, a.sb = sb, a.ldb = up(N, 16);
            a.B = nullptr, a.Bt = bt, a.ldbt = ldt;
            return launch_gemm_f8(cfg, a, vec8, s, config < 0);
        }
        const int64_t ldk = up(K, 16), ldn = up(N, 16);
        const int64_t cA = mfg_convert_bytes(M, K, ldk, MFG_FP8_E4M3), cB = mfg_convert_bytes(K, N, ldn, MFG_FP8_E4M3);
        CallWs ws;
        if ((st = call_ws(s, (size_t)(up(cA, 256) + up(cB, 256)), ext, ws)) != MFG_OK) return st;
        uint8_t* qa = static_cast<uint8_t*>(ws.ptr);
        uint8_t* qb = qa + up(cA, 256);
        float* sa = reinterpret_cast<float*>(qa + mfg_fp8_scale_offset(M, ldk));
        float* sb = reinterpret_cast<float*>(qb + mfg_fp8_scale_offset(K, ldn));
        const QuantJob ja{Af, qa, sa, M, K, lda, ldk, M, K, 0}, jb{Bf, qb, sb, K, N, ldb, ldn, K, N, 0};
        if ((st = launch_quantize_fp8_pair(ja, &jb, s)) != MFG_OK) return st;
        a.A = qa, a.lda = ldk, a.sa = sa, a.sb = sb, a.B = qb, a.ldb = ldn;
        return launch_gemm_f8(cfg, a, vec8, s);
    }

    if (m == MFG_BF16_SPLIT6) {
        // Both operands split three ways into the long-K layout (launch_split6_bf16),
        // then one BF16 GEMM over K' = 6 kp.
        if (pre) return MFG_ERR_UNSUPPORTED;
        const int64_t kp = up(K, 64), kk = 6 * kp, ldn = up(N, 8);
        const int64_t ea = up(M * kk, 128), eb = up(kk * ldn, 128);
        CallWs ws;
        if ((st = call_ws(s, (size_t)(ea + eb) * 2, ext, ws)) != MFG_OK) return st;
        uint16_t* a0 = static_cast<uint16_t*>(ws.ptr);
        uint16_t* b0 = a0 + ea;
        if ((st = launch_split6_bf16(M, K, static_cast<const float*>(A), lda, a0, kk, kp, false, s)) != MFG_OK)
            return st;
        if ((st = launch_split6_bf16(K, N, static_cast<const float*>(B), ldb, b0, ldn, kp, true, s)) != MFG_OK)
            return st;
        Gemm16Args a{};
        a.M = M, a.N = N, a.K = kk, a.C = C, a.ldc = ldc, a.alpha = alpha, a.beta = beta;
        a.A[0] = a0, a.B[0] = b0, a.lda = kk, a.ldb = ldn;
        const bool vec = buffer_ldc_ok(ldc) && operand_ld_ok(kk, ldn);
        const int cfg = choose_split6(config, M, N, K, ldc, vec);
        if (ran) *ran = cfg;
        return launch_gemm16(K_BF16, cfg, a, 1, vec, s, config < 0);
    }

    // 16-bit modes
    const int kind = kind_of(m);
    const int n16 = num_configs16(kind);  // configurations n16.. are the fused FP32-input kernels
    if (config >= n16 + num_configs_fused(kind)) return MFG_ERR_INVALID_ARG;
    if (!pre) {
        const FusedArgs fa{M, N, K, static_cast<const float*>(A), static_cast<const float*>(B), C, lda, ldb, ldc,
                           alpha, beta};
        int fc = config >= n16 ? config - n16 : -1;
        if (config < 0) {
            const int t = tuned(config, m, M, N, K);
            if (t >= n16 && fused_ok(kind, t - n16, fa)) fc = t - n16;
            // allocation-free call whose planes would not fit its array: the
            // fused kernel needs none
            const int64_t planes = (npa(m) * up(M * up(K, 8), 128) + npb(m) * up(K * up(N, 8), 128)) * 2;
            if (fc < 0 && ext && planes > (int64_t)ext->cap && fused_ok(kind, 0, fa)) fc = 0;
        }
        if (fc >= 0) {
            if (ran) *ran = n16 + fc;
            return launch_gemm_fused(kind, fc, fa, s);
        }
    } else if (config >= n16) {
        return MFG_ERR_UNSUPPORTED;  // the fused kernels read FP32 operands
    }
    Gemm16Args a{};
    a.M = M, a.N = N, a.K = K, a.C = C, a.ldc = ldc, a.alpha = alpha, a.beta = beta;
    if (pre) {
        const uint16_t* pa = static_cast<const uint16_t*>(A);
        const uint16_t* pb = static_cast<const uint16_t*>(B);
        a.A[0] = pa, a.A[1] = npa(m) == 2 ? pa + M * lda : nullptr;
        a.B[0] = pb, a.B[1] = npb(m) == 2 ? pb + K * ldb : nullptr;
        a.lda = lda, a.ldb = ldb;
        const bool vec =
            al16(A) && al16(B) && lda % 8 == 0 && ldb % 8 == 0 && buffer_ldc_ok(ldc) && operand_ld_ok(lda, ldb);
        const int cfg = choose16(m, config, M, N, K, K, ldc, vec);
        if (ran) *ran = cfg;
        return launch_gemm16(kind, cfg, a, 1, vec, s, config < 0);
    }
    const auto [kp, ldk, ldn] = planes16(M, N, K, ext != nullptr);
    const int64_t pa_elems = M * ldk, pb_elems = kp * ldn;
    const size_t bytes = (size_t)(npa(m) * up(pa_elems, 128) + npb(m) * up(pb_elems, 128)) * 2;
    CallWs ws;
    if ((st = call_ws(s, bytes, ext, ws)) != MFG_OK) return st;
    uint16_t* w = static_cast<uint16_t*>(ws.ptr);
    uint16_t* a0 = w;
    uint16_t* a1 = npa(m) == 2 ? a0 + up(pa_elems, 128) : nullptr;
    uint16_t* b0 = (a1 ? a1 : a0) + up(pa_elems, 128);
    uint16_t* b1 = npb(m) == 2 ? b0 + up(pb_elems, 128) : nullptr;
    if ((st = convert16_pair(m, M, N, K, kp, static_cast<const float*>(A), lda, static_cast<const float*>(B), ldb, a0, a1,
                             ldk, b0, b1, ldn, s)) != MFG_OK)
        return st;
    a.K = kp;
    a.A[0] = a0, a.A[1] = a1, a.B[0] = b0, a.B[1] = b1, a.lda = ldk, a.ldb = ldn;
    const bool vec = buffer_ldc_ok(ldc) && operand_ld_ok(ldk, ldn);  // workspace planes: aligned, ld a multiple of 8
    const int cfg = choose16(m, config, M, N, K, kp, ldc, vec);
    if (config >= 0 && !config16_ok(kind, cfg, M, N, K, ldc, vec)) return MFG_ERR_UNSUPPORTED;  // judged on the caller's K
    if (ran) *ran = cfg;
    return launch_gemm16(kind, cfg, a, 1, vec, s, config < 0);
}

}  // namespace mfg

using namespace mfg;

#define MFG_GUARD(expr)                      \
    try {                                    \
        return (expr);                       \
    } catch (const std::bad_alloc&) {        \
        return MFG_ERR_NO_MEMORY;            \
    } catch (...) {                          \
        return MFG_ERR_INTERNAL;             \
    }

extern "C" int mfg_gemm(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                        float* C, int64_t ldc, float alpha, float beta, int mode, void* stream) {
    MFG_GUARD(gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, mode, -1, (hipStream_t)stream));
}

// Scratch of the allocation-free entry point (noalloc.hip): this device's
// copy of the array and its size.
namespace mfg {
int noalloc_scratch(void** ptr, size_t* bytes);
}

extern "C" int mfg_gemm_noalloc(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                                int64_t ldb, float* C, int64_t ldc, float alpha, float beta, int mode, void* stream) {
    try {
        int st = validate_gemm(M, N, K, A, lda, B, ldb, C, ldc, mode);
        if (st != MFG_OK) return st;
        ExtWs ext{nullptr, 0};
        if ((st = noalloc_scratch(&ext.ptr, &ext.cap)) != MFG_OK) return st;
        return gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, mode, -1, (hipStream_t)stream, &ext);
    } catch (const std::bad_alloc&) {
        return MFG_ERR_NO_MEMORY;
    } catch (...) {
        return MFG_ERR_INTERNAL;
    }
}

extern "C" int mfg_gemm_config(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                               int64_t ldb, float* C, int64_t ldc, float alpha, float beta, int mode, int config,
                               void* stream) {
    if (config < -1) return MFG_ERR_INVALID_ARG;
    MFG_GUARD(gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, mode, config, (hipStream_t)stream));
}

extern "C" int mfg_num_configs(int mode) {
    int m = mode & MFG_MODE_MASK;
    if (m == MFG_BF16_SPLIT6) m = MFG_BF16;  // runs the BF16 kernels
    if (m == MFG_F32) return num_configs_f32();
    if (m == MFG_FP8_E4M3) return num_configs_f8();
    const int k = kind_of(m);
    return k < 0 ? MFG_ERR_INVALID_ARG : num_configs16(k) + num_configs_fused(k);
}

extern "C" int mfg_config_name(int mode, int config, char* buf, int n) {
    int m = mode & MFG_MODE_MASK;
    if (m == MFG_BF16_SPLIT6) m = MFG_BF16;
    const char* name = nullptr;
    if (m == MFG_F32) name = config_f32_name(config);
    else if (m == MFG_FP8_E4M3) name = config_f8_name(config);
    else if (kind_of(m) >= 0) {
        const int k = kind_of(m), n16 = num_configs16(k);
        name = config < n16 ? config16_name(k, config) : config_fused_name(k, config - n16);
    }
    if (!name || !buf || n <= 0) return MFG_ERR_INVALID_ARG;
    std::strncpy(buf, name, (size_t)n - 1);
    buf[n - 1] = '\0';
    return MFG_OK;
}

extern "C" int mfg_tune_lookup(int64_t M, int64_t N, int64_t K, int mode) {
    const int m = mode & MFG_MODE_MASK;
    if (m < 0 || m >= MFG_NUM_MODES || M < 0 || N < 0 || K < 0) return MFG_ERR_INVALID_ARG;
    // as gemm_impl chooses, for contiguous operands (preconverted: ld rounded up
    // to whole 16-byte pieces)
    const bool pre = (mode & MFG_IN_PRECONVERTED) != 0, cbuf = buffer_ldc_ok(N);
    const int t = tuned_lookup(m, M, N, K);
    if (m == MFG_F32) {
        const bool vec = K % 4 == 0 && N % 4 == 0;
        return (t >= 0 && config_f32_ok(t, N, vec)) ? t : cbuf ? pick_config_f32(M, N, K, vec) : 0;
    }
    if (m == MFG_FP8_E4M3) {
        const bool vec = cbuf && up(K, 128) < kF8LdLimit;
        return (t >= 0 && config_f8_ok(t, M, N, K, N, vec)) ? t : pick_config_f8(M, N, K, vec, pre);
    }
    if (m == MFG_BF16_SPLIT6) return choose_split6(-1, M, N, K, N, cbuf && operand_ld_ok(6 * up(K, 64), up(N, 8)));
    if (pre) return choose16(m, -1, M, N, K, K, N, cbuf && operand_ld_ok(up(K, 8), up(N, 8)));
    // FP32 operands: a tuned fused kernel where the shape allows it
    const int k = kind_of(m), n16 = num_configs16(k);
    if (t >= n16 && t < n16 + num_configs_fused(k) && K % 64 == 0 && K > 0 && N % 8 == 0 && N >= 8 && M >= 1) return t;
    const Planes16 p = planes16(M, N, K, false);
    return choose16(m, -1, M, N, K, p.kp, N, cbuf && operand_ld_ok(p.ldk, p.ldn));
}

// -------------------------------------------------------------------- batched
static int batched_impl(int64_t count, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                        int64_t strideA, const void* B, int64_t ldb, int64_t strideB, float* C, int64_t ldc,
                        int64_t strideC, float alpha, float beta, int mode, hipStream_t s) {
    const int m = mode & MFG_MODE_MASK;
    // Only MFG_IN_PRECONVERTED may accompany the mode (validate_gemm checks
    // the flags).  F16 / BF16 / F32 take their operands as stored, so the
    // flag is implied there; the refined modes read each entry in its
    // preconverted form with it, and FP32 operands without it.
    const bool pre = (mode & MFG_IN_PRECONVERTED) != 0;
    if (count < 0 || strideA < 0 || strideB < 0 || strideC < 0) return MFG_ERR_INVALID_ARG;
    int st = validate_gemm(M, N, K, A, lda, B, ldb, C, ldc, mode);
    if (st != MFG_OK) return st;
    if (count > 1 && M > 0 && N > 0 && strideC < (M - 1) * ldc + N) return MFG_ERR_INVALID_ARG;  // outputs overlap
    if (m == MFG_FP8_E4M3 || m == MFG_BF16_SPLIT6) return MFG_ERR_UNSUPPORTED;
    if (count == 0 || M == 0 || N == 0) return MFG_OK;
    if (K == 0 || alpha == 0.0f) return launch_scale_c(M, N, C, ldc, beta, count, strideC, s);

    if (m == MFG_F32) {
        GemmF32Args a{};
        a.M = M, a.N = N, a.K = K, a.ldc = ldc, a.alpha = alpha, a.beta = beta;
        a.lda = lda, a.ldb = ldb, a.sA = strideA, a.sB = strideB, a.sC = strideC;
        const bool vec = al16(A) && al16(B) && lda % 4 == 0 && ldb % 4 == 0 && strideA % 4 == 0 && strideB % 4 == 0 &&
                         buffer_ldc_ok(ldc);
        const int cfg = buffer_ldc_ok(ldc) ? pick_config_f32(M, N, K, vec && K % 4 == 0, count) : 0;
        for (int64_t b0 = 0; b0 < count; b0 += 65535) {
            a.A = static_cast<const float*>(A) + b0 * strideA;
            a.B = static_cast<const float*>(B) + b0 * strideB;
            a.C = C + b0 * strideC;
            if ((st = launch_gemm_f32(cfg, a, std::min<int64_t>(65535, count - b0), vec, s, true)) != MFG_OK) return st;
        }
        return MFG_OK;
    }

    const int kind = kind_of(m);
    Gemm16Args a{};
    a.M = M, a.N = N, a.K = K, a.C = C, a.ldc = ldc, a.sC = strideC, a.alpha = alpha, a.beta = beta;
    bool vec;
    const bool split_mode = two_planes_a(m);
    std::unique_ptr<WsLease> ws;
    if (split_mode && pre) {
        // entry b: head plane at A + b*strideA, residual plane rows*ld later
        const uint16_t* pa = static_cast<const uint16_t*>(A);
        const uint16_t* pb = static_cast<const uint16_t*>(B);
        a.A[0] = pa, a.A[1] = pa + M * lda;
        a.B[0] = pb, a.B[1] = two_planes_b(m) ? pb + K * ldb : nullptr;
        a.lda = lda, a.ldb = ldb, a.sA = strideA, a.sB = strideB;
        vec = al16(A) && al16(B) && lda % 8 == 0 && ldb % 8 == 0 && strideA % 8 == 0 && strideB % 8 == 0 &&
              buffer_ldc_ok(ldc) && operand_ld_ok(lda, ldb);
    } else if (!split_mode) {
        a.A[0] = static_cast<const uint16_t*>(A), a.B[0] = static_cast<const uint16_t*>(B);
        a.lda = lda, a.ldb = ldb, a.sA = strideA, a.sB = strideB;
        vec = al16(A) && al16(B) && lda % 8 == 0 && ldb % 8 == 0 && strideA % 8 == 0 && strideB % 8 == 0 &&
              buffer_ldc_ok(ldc) && operand_ld_ok(lda, ldb);
    } else {
        // FP32 operands split into the workspace, packed per batch entry.
        const int64_t ldk = up(K, 8), ldn = up(N, 8);
        const int64_t pa = up(M * ldk, 8), pb = up(K * ldn, 8);
        const size_t bytes = (size_t)(npa(m) * count * pa + npb(m) * count * pb) * 2 + 1024;
        ws.reset(new WsLease(s, bytes));
        if (!ws->ptr()) return ws->status();
        uint16_t* w = static_cast<uint16_t*>(ws->ptr());
        uint16_t* a0 = w;
        uint16_t* a1 = a0 + count * pa;
        uint16_t* b0 = a1 + count * pa;
        uint16_t* b1 = npb(m) == 2 ? b0 + count * pb : nullptr;
        const float* Af = static_cast<const float*>(A);
        const float* Bf = static_cast<const float*>(B);
        // A contiguous batch (stride == rows * ld) is one tall matrix.
        const bool tall_a = strideA == M * lda && pa == M * ldk, tall_b = strideB == K * ldb && pb == K * ldn;
        const bool bsplit = npb(m) == 2;  // REFINE_A: B rounded to its FP16 head only
        st = MFG_ERR_UNSUPPORTED;
        if (tall_a && tall_b)
            st = launch_convert_pair(ConvJob{Af, a0, lda, ldk, count * M, K, count * M, K, a1 - a0, conv_kind(m, true), 0},
                                     ConvJob{Bf, b0, ldb, ldn, count * K, N, count * K, N, bsplit ? b1 - b0 : 0, conv_kind(m, bsplit), 0},
                                     s);
        if (st != MFG_OK && st != MFG_ERR_UNSUPPORTED) return st;
        if (st == MFG_ERR_UNSUPPORTED) {
            if (tall_a) {
                if ((st = convert16(m, count * M, K, Af, lda, a0, a1, ldk, true, s)) != MFG_OK) return st;
            } else {
                for (int64_t b = 0; b < count; ++b)
                    if ((st = convert16(m, M, K, Af + b * strideA, lda, a0 + b * pa, a1 + b * pa, ldk, true, s)) != MFG_OK)
                        return st;
            }
            if (tall_b) {
                if ((st = convert16(m, count * K, N, Bf, ldb, b0, b1, ldn, bsplit, s)) != MFG_OK) return st;
            } else {
                for (int64_t b = 0; b < count; ++b)
                    if ((st = convert16(m, K, N, Bf + b * strideB, ldb, b0 + b * pb, bsplit ? b1 + b * pb : nullptr, ldn,
                                        bsplit, s)) != MFG_OK)
                        return st;
            }
        }
        a.A[0] = a0, a.A[1] = a1, a.B[0] = b0, a.B[1] = b1;
        a.lda = ldk, a.ldb = ldn, a.sA = pa, a.sB = pb;
        vec = buffer_ldc_ok(ldc) && operand_ld_ok(ldk, ldn);
    }
    if (M <= 32 && N <= 32) return launch_batched_small(kind, a, count, vec, device_cu_count(), s);
    const int cfg = vec ? pick_config16(kind, M, N, K, vec, count) : 0;
    for (int64_t b0 = 0; b0 < count; b0 += 65535) {
        Gemm16Args c = a;
        for (int q = 0; q < 2; ++q) {
            if (c.A[q]) c.A[q] += b0 * a.sA;
            if (c.B[q]) c.B[q] += b0 * a.sB;
        }
        c.C = C + b0 * strideC;
        if ((st = launch_gemm16(kind, cfg, c, std::min<int64_t>(65535, count - b0), vec, s, true)) != MFG_OK) return st;
    }
    return MFG_OK;
}

extern "C" int mfg_gemm_batched(int64_t count, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                                int64_t strideA, const void* B, int64_t ldb, int64_t strideB, float* C, int64_t ldc,
                                int64_t strideC, float alpha, float beta, int mode, void* stream) {
    MFG_GUARD(batched_impl(count, M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, alpha, beta, mode,
                           (hipStream_t)stream));
}

// -------------------------------------------------------------------- grouped
// Largest M or N of a plan whose FP32 operands the grouped kernel may convert
// itself (pass and kernel -> kernel alone: 64 of 1024^3 F16 375 -> 397 us, 16 of
// 2048^3 SPLIT3 1557 -> 1710, F16 569 -> 658).
constexpr int64_t kGroupedDirect = 768;

struct mfg_grouped_plan {
    int mode = 0, kind = 0, device = 0;
    int64_t count = 0, nwork = 0;
    // tile classes present in the plan: work items of class c are the range
    // split[c] of the one work array (one launch per class)
    int nclass = 0;
    int tile[2] = {0, 0};
    GroupedSplit split[2]{};
    GroupedWork* d_work = nullptr;
    int64_t* d_planes = nullptr;  // refined modes: residual-plane offsets per work item
    // MFG_IN_FP32: converted operands (plan-owned) and the conversion job list
    void* d_conv = nullptr;
    ConvJob* d_jobs = nullptr;
    ConvTask* d_tasks = nullptr;
    int64_t ntasks = 0;
    bool f32 = false;  // MFG_IN_FP32 with the conversion in the grouped kernel: none of the four above
    double flops = 0.0, bytes = 0.0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    float g_alpha = 0.f, g_beta = 0.f;
    hipStream_t cap_stream = nullptr;  // capture happens here: the legacy NULL stream cannot be captured
};

static void plan_free(mfg_grouped_plan* plan) {
    if (plan->exec) (void)hipGraphExecDestroy(plan->exec);
    if (plan->graph) (void)hipGraphDestroy(plan->graph);
    if (plan->d_work) (void)hipFree(plan->d_work);
    if (plan->d_planes) (void)hipFree(plan->d_planes);
    if (plan->d_conv) (void)hipFree(plan->d_conv);
    if (plan->d_jobs) (void)hipFree(plan->d_jobs);
    if (plan->d_tasks) (void)hipFree(plan->d_tasks);
    if (plan->cap_stream) (void)hipStreamDestroy(plan->cap_stream);
    delete plan;
}

// Host array -> new device allocation (nullptr for an empty array).
template <class T>
static int upload(const std::vector<T>& h, T** d) {
    *d = nullptr;
    if (h.empty()) return MFG_OK;
    if (hipMalloc((void**)d, h.size() * sizeof(T)) != hipSuccess) {
        *d = nullptr;
        (void)hipGetLastError();
        return MFG_ERR_NO_MEMORY;
    }
    MFG_HIP_CHECK(hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
    return MFG_OK;
}

// The tile class a problem of mode m runs in: its size bucket's tuned entry
// if there is a valid one, else the kind's default; `force` (> 0) overrides.
static int grouped_class(int m, int kind, int64_t M, int64_t N, int64_t K, int force) {
    if (force > 0) return force;
    const int t = tuned_lookup(kGroupedTuneBase + m, M, N, K);
    return (t > 0 && grouped_tile_ok(kind, t)) ? t : grouped_tile(kind);
}

// Whether a plan's FP32 operands are converted in the grouped kernel instead
// of by a pass before it, where that costs less.  The pass is a launch (3.5 us)
// and 6 or 8 bytes per element at the copy rate.  In the kernel every tile that
// reads an element converts it: per 64-deep block of K that adds to the tile's
// chain of loads and stores, 0.55 us to a 128 x 128 tile (1.25 past K = 4096) and
// 0.27 to a 64 x 64 tile, or, with many tiles, their sum over the CUs, 0.8 and
// 0.16 (REFINE_A 1.43 times that past sides of 512).  us, with pass and without,
// SPLIT3 and F16: 4096 problems of 128^3 356 -> 174 and 251 -> 160, 256 of 512^3
// 586 -> 483 and 283 -> 235, 128 of 768^3 848 -> 796 and 375 -> 342; a long K or
// few tiles are the other way round: F16 4 of 128 x 128 x 32768 517 and 761, one
// of 256 x 256 x 2048 38 and 47, 18 of 768 x 768 x 8192 559 and 643 (of 280 plans
// the choice costs 0.1% on average, the kernel alone 9.5%, the pass alone 11.7%).
// Only without a C that overlaps an operand: the pass reads all of them before
// any C is written.
static bool grouped_converts(int64_t count, const mfg_problem* probs, int m, int force_tile) {
    const int kind = kind_of(m);
    const double planes_a = two_planes_a(m) ? 2.0 : 1.0, planes_b = two_planes_b(m) ? 2.0 : 1.0;
    double bytes = 0.0, chain = 0.0, sum = 0.0, longest = 0.0;
    for (int64_t i = 0; i < count; ++i) {
        const mfg_problem& p = probs[i];
        const int tile = grouped_class(m, kind, p.M, p.N, p.K, force_tile);
        const double tiles = (double)(cdiv(p.M, tile) * cdiv(p.N, tile)), blocks = (double)cdiv(p.K, 64);
        bytes += (double)(p.M * p.K) * (4.0 + 2.0 * planes_a) + (double)(p.K * p.N) * (4.0 + 2.0 * planes_b);
        if (tiles == 0.0) continue;
        double each = tile == 128 ? 0.8 : 0.16, link = tile == 128 ? (p.K > 4096 ? 1.25 : 0.55) : 0.27;
        if (planes_a != planes_b && (p.M > 512 || p.N > 512)) each *= 1.43, link *= 1.43;
        sum += each * tiles * blocks / 256.0;
        longest = std::max(longest, (tile == 128 ? 0.5 : 1.0) * each * blocks);
        chain = std::max(chain, link * blocks);
    }
    return std::max(chain, sum + longest) < 3.5 + bytes / 5.3e6;
}

static bool grouped_direct(int64_t count, const mfg_problem* probs, int m, int force_tile) {
    if (!grouped_converts(count, probs, m, force_tile)) return false;
    struct Range {
        uintptr_t lo, hi;
    };
    std::vector<Range> in, out;
    auto add = [](std::vector<Range>& v, const void* p, int64_t rows, int64_t cols, int64_t ld) {
        if (rows > 0 && cols > 0)
            v.push_back({(uintptr_t)p, (uintptr_t)p + (size_t)((rows - 1) * ld + cols) * sizeof(float)});
    };
    for (int64_t i = 0; i < count; ++i) {
        const mfg_problem& p = probs[i];
        if (p.M > kGroupedDirect || p.N > kGroupedDirect || !buffer_ldc_ok(p.ldc) || !operand_ld_ok(p.lda, p.ldb)) return false;
        if (((uintptr_t)p.A | (uintptr_t)p.B) % sizeof(float) != 0) return false;
        add(in, p.A, p.M, p.K, p.lda), add(in, p.B, p.K, p.N, p.ldb), add(out, p.C, p.M, p.N, p.ldc);
    }
    auto by_lo = [](const Range& a, const Range& b) { return a.lo < b.lo; };
    std::sort(in.begin(), in.end(), by_lo);
    std::sort(out.begin(), out.end(), by_lo);
    // each operand against the outputs that start before its end: the furthest end of those
    uintptr_t reach = 0;
    size_t c = 0;
    for (const Range& r : in) {
        for (; c < out.size() && out[c].lo <= r.lo; ++c) reach = std::max(reach, out[c].hi);
        if (reach > r.lo || (c < out.size() && out[c].lo < r.hi)) return false;
    }
    return true;
}

static int plan_create_impl(int64_t count, const mfg_problem* probs, int mode, mfg_grouped_plan** out,
                            int force_tile = 0) {
    if (!out || count < 0 || (count > 0 && !probs)) return MFG_ERR_INVALID_ARG;
    *out = nullptr;
    const int m = mode & MFG_MODE_MASK;
    if ((mode & ~(MFG_MODE_MASK | MFG_IN_PRECONVERTED | MFG_IN_FP32)) != 0 || m < 0 || m >= MFG_NUM_MODES)
        return MFG_ERR_INVALID_ARG;
    const bool fp32_in = (mode & MFG_IN_FP32) != 0;
    if (fp32_in && (mode & MFG_IN_PRECONVERTED)) return MFG_ERR_INVALID_ARG;
    if (m == MFG_F32 || m == MFG_FP8_E4M3 || m == MFG_BF16_SPLIT6) return MFG_ERR_UNSUPPORTED;
    if (count > ((int64_t)1 << 31) - 1) return MFG_ERR_UNSUPPORTED;
    // Refined modes read their operands in the preconverted storage form:
    // A's residual plane at A + M*lda, and for the two-sided splits B's at
    // B + K*ldb.
    const bool two_a = two_planes_a(m), two_b = two_planes_b(m);
    std::vector<GroupedDesc> descs((size_t)count);
    std::vector<GroupedWork> work;
    double flops = 0.0, bytes = 0.0;
    bool direct = fp32_in;  // (decided once the arguments are checked)
    for (int64_t i = 0; i < count && fp32_in; ++i) {
        const mfg_problem& p = probs[i];
        const int st = validate_gemm(p.M, p.N, p.K, p.A, p.lda, p.B, p.ldb, p.C, p.ldc, m);
        if (st != MFG_OK) return st;
        if (p.M > ((int64_t)1 << 24) || p.N > ((int64_t)1 << 24) || p.K > INT32_MAX) return MFG_ERR_UNSUPPORTED;
    }
    direct = direct && grouped_direct(count, probs, m, force_tile);
    // MFG_IN_FP32: byte offsets of each problem's converted A and B in the
    // plan's storage (256-byte aligned, ld rounded up to 8 elements)
    std::vector<int64_t> conv_off(fp32_in ? (size_t)count * 2 : 0);
    int64_t conv_bytes = 0;
    for (int64_t i = 0; i < count; ++i) {
        const mfg_problem& p = probs[i];
        int st = validate_gemm(p.M, p.N, p.K, p.A, p.lda, p.B, p.ldb, p.C, p.ldc, m);
        if (st != MFG_OK) return st;
        if (p.M > ((int64_t)1 << 24) || p.N > ((int64_t)1 << 24) || p.K > INT32_MAX) return MFG_ERR_UNSUPPORTED;
        GroupedDesc& d = descs[(size_t)i];
        d.M = p.M, d.N = p.N, d.K = p.K, d.ldc = p.ldc, d.C = p.C, d.pad = 0;
        if (fp32_in) {  // A and B point into the plan's storage once it exists
            d.lda = up(p.K, 8), d.ldb = up(p.N, 8), d.vec = 1;
            conv_off[2 * i] = conv_bytes;
            conv_bytes += up((two_a ? 2 : 1) * p.M * d.lda * 2, 256);
            conv_off[2 * i + 1] = conv_bytes;
            conv_bytes += up((two_b ? 2 : 1) * p.K * d.ldb * 2, 256);
            bytes += 4.0 * (double)(p.M * p.K + p.K * p.N) +
                     2.0 * ((two_a ? 2.0 : 1.0) * (double)(p.M * p.K) + (two_b ? 2.0 : 1.0) * (double)(p.K * p.N));
        } else {
            d.lda = p.lda, d.ldb = p.ldb;
            d.A = static_cast<const uint16_t*>(p.A), d.B = static_cast<const uint16_t*>(p.B);
            d.vec = (al16(p.A) && al16(p.B) && p.lda % 8 == 0 && p.ldb % 8 == 0) ? 1 : 0;
        }
        if (direct) {
            d.lda = p.lda, d.ldb = p.ldb;
            d.A = static_cast<const uint16_t*>(p.A), d.B = static_cast<const uint16_t*>(p.B);
        }
        d.pa = two_a ? p.M * d.lda : 0;
        d.pb = two_b ? p.K * d.ldb : 0;
        flops += 2.0 * (double)p.M * (double)p.N * (double)p.K;
        bytes += 2.0 * ((two_a ? 2.0 : 1.0) * (double)(p.M * p.K) + (two_b ? 2.0 : 1.0) * (double)(p.K * p.N)) +
                 4.0 * (double)(p.M * p.N);
    }
    std::unique_ptr<mfg_grouped_plan, void (*)(mfg_grouped_plan*)> plan(new mfg_grouped_plan(), plan_free);
    plan->mode = m, plan->kind = kind_of(m), plan->count = count;
    plan->flops = flops, plan->bytes = bytes;
    MFG_HIP_CHECK(hipGetDevice(&plan->device));
    plan->f32 = direct;
    if (fp32_in && !direct && conv_bytes > 0) {
        if (hipMalloc(&plan->d_conv, (size_t)conv_bytes) != hipSuccess) {
            plan->d_conv = nullptr;
            (void)hipGetLastError();
            return MFG_ERR_NO_MEMORY;
        }
        // conversion jobs (A then B of every problem) and their row tasks
        std::vector<ConvJob> jobs;
        std::vector<ConvTask> tasks;
        char* base = static_cast<char*>(plan->d_conv);
        for (int64_t i = 0; i < count; ++i) {
            const mfg_problem& p = probs[i];
            GroupedDesc& d = descs[(size_t)i];
            d.A = reinterpret_cast<const uint16_t*>(base + conv_off[2 * i]);
            d.B = reinterpret_cast<const uint16_t*>(base + conv_off[2 * i + 1]);
            const ConvJob ja{static_cast<const float*>(p.A), const_cast<uint16_t*>(d.A), p.lda, d.lda, p.M, p.K,
                             p.M, p.K, d.pa, conv_kind(m, two_a), conv_rows_per_task(p.M, p.K)};
            const ConvJob jb{static_cast<const float*>(p.B), const_cast<uint16_t*>(d.B), p.ldb, d.ldb, p.K, p.N,
                             p.K, p.N, d.pb, conv_kind(m, two_b), conv_rows_per_task(p.K, p.N)};
            for (const ConvJob& j : {ja, jb}) {
                if (j.rows == 0 || j.cols == 0) continue;
                if ((int64_t)jobs.size() >= INT32_MAX) return MFG_ERR_UNSUPPORTED;
                const int32_t ji = (int32_t)jobs.size();
                jobs.push_back(j);
                for (int64_t r = 0; r < j.rows; r += j.rpt) tasks.push_back(ConvTask{ji, (int32_t)r});
            }
        }
        int st = upload(jobs, &plan->d_jobs);
        if (st == MFG_OK) st = upload(tasks, &plan->d_tasks);
        if (st != MFG_OK) return st;
        plan->ntasks = (int64_t)tasks.size();
    }
    // problems by tile class, then one work list per class, concatenated
    const int kind = kind_of(m);
    if (force_tile > 0 && !grouped_tile_ok(kind, force_tile)) return MFG_ERR_UNSUPPORTED;
    int tiles[2];
    const int ntiles = grouped_tiles(kind, tiles);
    // Each class is one more launch with its own tail: a class carrying under
    // a quarter of the plan's flops runs in the other one instead.
    std::vector<int> cls((size_t)count);
    double cflops[2] = {0.0, 0.0};
    for (int64_t i = 0; i < count; ++i) {
        const GroupedDesc& d = descs[(size_t)i];
        cls[(size_t)i] = grouped_class(m, kind, d.M, d.N, d.K, force_tile);
        cflops[cls[(size_t)i] == tiles[0] ? 0 : 1] += 2.0 * (double)d.M * (double)d.N * (double)d.K;
    }
    if (ntiles == 2 && cflops[0] > 0.0 && cflops[1] > 0.0) {
        const int minor = cflops[0] < cflops[1] ? 0 : 1;
        if (cflops[minor] < 0.25 * (cflops[0] + cflops[1]))
            for (int& c : cls) c = tiles[1 - minor];
    }
    std::vector<int64_t> planes;
    for (int c = 0; c < ntiles; ++c) {
        std::vector<GroupedDesc> sub;
        for (int64_t i = 0; i < count; ++i)
            if (cls[(size_t)i] == tiles[c]) sub.push_back(descs[(size_t)i]);
        if (sub.empty()) continue;
        std::vector<GroupedWork> w;
        std::vector<int64_t> pl;
        GroupedSplit sp{};
        build_grouped_work(sub.data(), (int64_t)sub.size(), w, sp, two_a && !direct ? &pl : nullptr, tiles[c],
                           direct ? 4 : 2);
        const int64_t base = (int64_t)work.size();
        for (auto& o : sp.off)
            for (auto& v : o) v += base;
        const int k = plan->nclass++;
        plan->tile[k] = tiles[c], plan->split[k] = sp;
        work.insert(work.end(), w.begin(), w.end());
        planes.insert(planes.end(), pl.begin(), pl.end());
    }
    plan->nwork = (int64_t)work.size();
    int st = upload(work, &plan->d_work);
    if (st == MFG_OK && two_a && !direct) st = upload(planes, &plan->d_planes);
    if (st != MFG_OK) return st;
    *out = plan.release();
    return MFG_OK;
}

// One run of a plan on stream s: the conversion pass (MFG_IN_FP32), then the
// grouped kernel launch(es).
static int plan_launch(mfg_grouped_plan* plan, float alpha, float beta, hipStream_t s) {
    if (plan->ntasks > 0) {
        const int st = launch_convert_jobs(plan->d_jobs, plan->d_tasks, plan->ntasks, s);
        if (st != MFG_OK) return st;
    }
    for (int c = 0; c < plan->nclass; ++c) {
        const int st = grouped_launch(plan->kind, plan->tile[c], plan->d_work, plan->d_planes, plan->split[c], alpha,
                                      beta, s, plan->f32);
        if (st != MFG_OK) return st;
    }
    return MFG_OK;
}

extern "C" int mfg_grouped_plan_create(int64_t count, const mfg_problem* problems, int mode,
                                       mfg_grouped_plan** out) {
    MFG_GUARD(plan_create_impl(count, problems, mode, out));
}

// Time the grouped kernel on the caller's problems with every tile class of
// the mode forced on all of them (alpha = 1, beta = 0: C is output only),
// check each class's outputs bitwise against the first class's, and record
// the fastest for the size bucket of the first problem.
static int grouped_autotune_impl(int64_t count, const mfg_problem* probs, int mode, int reps, int* best_tile,
                                 float* best_ms, hipStream_t s) {
    if (count < 1 || !probs || reps < 1) return MFG_ERR_INVALID_ARG;
    const int m = mode & MFG_MODE_MASK;
    if (m < 0 || m >= MFG_NUM_MODES || kind_of(m) < 0 || m == MFG_BF16_SPLIT6) return MFG_ERR_UNSUPPORTED;
    const int kind = kind_of(m);
    int tiles[2];
    const int ntiles = grouped_tiles(kind, tiles);
    int64_t total = 0;
    std::vector<int64_t> roff((size_t)count);
    for (int64_t i = 0; i < count; ++i) {
        if (probs[i].M < 0 || probs[i].N < 0) return MFG_ERR_INVALID_ARG;
        roff[(size_t)i] = total;
        total += probs[i].M * probs[i].N;
    }
    float* ref = nullptr;
    unsigned long long* cnt = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    mfg_grouped_plan* plan = nullptr;
    auto cleanup = [&]() {
        if (plan) plan_free(plan);
        if (ref) (void)hipFree(ref);
        if (cnt) (void)hipFree(cnt);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    if (hipMalloc(&ref, (size_t)std::max<int64_t>(total, 1) * sizeof(float)) != hipSuccess ||
        hipMalloc(&cnt, (size_t)count * sizeof(unsigned long long)) != hipSuccess) {
        (void)hipGetLastError();
        cleanup();
        return MFG_ERR_NO_MEMORY;
    }
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        cleanup();
        return MFG_ERR_HIP;
    }
    int st = MFG_OK, best = 0;
    float bms = 3.4e38f;
    std::vector<unsigned long long> bad((size_t)count);
    for (int c = 0; c < ntiles && st == MFG_OK; ++c) {
        if (plan) plan_free(plan), plan = nullptr;
        st = plan_create_impl(count, probs, mode, &plan, tiles[c]);
        if (st != MFG_OK) break;
        st = plan_launch(plan, 1.f, 0.f, s);  // warm-up, and the outputs checked below
        float total_ms = 0.f;
        for (int r = 0; r < reps && st == MFG_OK; ++r) {
            if (hipEventRecord(e0, s) != hipSuccess) st = MFG_ERR_HIP;
            if (st == MFG_OK) st = plan_launch(plan, 1.f, 0.f, s);
            if (st == MFG_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess))
                st = MFG_ERR_HIP;
            float ms = 0.f;
            if (st == MFG_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = MFG_ERR_HIP;
            total_ms += ms;
        }
        for (int64_t i = 0; i < count && st == MFG_OK; ++i) {
            const mfg_problem& p = probs[i];
            if (p.M == 0 || p.N == 0) continue;
            float* r = ref + roff[(size_t)i];
            if (c == 0) {
                if (hipMemcpy2DAsync(r, (size_t)p.N * 4, p.C, (size_t)p.ldc * 4, (size_t)p.N * 4, (size_t)p.M,
                                     hipMemcpyDeviceToDevice, s) != hipSuccess)
                    st = MFG_ERR_HIP;
            } else {
                st = launch_count_mismatch(p.M, p.N, static_cast<const float*>(p.C), p.ldc, r, p.N, cnt + i, s);
            }
        }
        if (st != MFG_OK) break;
        bool same = true;
        if (c > 0) {
            if (hipMemcpyAsync(bad.data(), cnt, (size_t)count * sizeof(unsigned long long), hipMemcpyDeviceToHost,
                               s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                st = MFG_ERR_HIP;
                break;
            }
            for (int64_t i = 0; i < count; ++i)
                if (probs[i].M > 0 && probs[i].N > 0 && bad[(size_t)i] != 0) same = false;
        }
        const float avg = total_ms / reps;
        if (same && avg < bms) bms = avg, best = tiles[c];
    }
    cleanup();
    if (st != MFG_OK) return st;
    for (int64_t i = 0; i < count; ++i) tuned_store(kGroupedTuneBase + m, probs[i].M, probs[i].N, probs[i].K, best);
    if (best_tile) *best_tile = best;
    if (best_ms) *best_ms = bms;
    return MFG_OK;
}

extern "C" int mfg_grouped_autotune(int64_t count, const mfg_problem* problems, int mode, int reps, int* best_tile,
                                    float* best_ms, void* stream) {
    MFG_GUARD(grouped_autotune_impl(count, problems, mode, reps, best_tile, best_ms, (hipStream_t)stream));
}

// The tile classes a plan launches and their work items.
extern "C" int mfg_grouped_plan_classes(const mfg_grouped_plan* plan, int* tiles, int64_t* items, int max) {
    if (!plan || max < 0 || (max > 0 && (!tiles || !items))) return MFG_ERR_INVALID_ARG;
    for (int c = 0; c < plan->nclass && c < max; ++c) {
        tiles[c] = plan->tile[c];
        items[c] = plan->split[c].off[0][kXcds] - plan->split[c].off[0][0] + plan->split[c].off[1][kXcds] -
                   plan->split[c].off[1][0];
    }
    return plan->nclass;
}

// Tile classes of a mode's grouped kernel (sides, the default first).
extern "C" int mfg_grouped_tile_classes(int mode, int* tiles, int max) {
    const int m = mode & MFG_MODE_MASK;
    if (!tiles || max < 1 || m < 0 || m >= MFG_NUM_MODES) return MFG_ERR_INVALID_ARG;
    const int kind = kind_of(m);
    if (kind < 0 || m == MFG_BF16_SPLIT6) return MFG_ERR_UNSUPPORTED;
    int t[2];
    const int n = grouped_tiles(kind, t);
    for (int i = 0; i < n && i < max; ++i) tiles[i] = t[i];
    return n;
}

extern "C" int mfg_grouped_run(mfg_grouped_plan* plan, float alpha, float beta, void* stream) {
    if (!plan) return MFG_ERR_INVALID_ARG;
    MFG_GUARD(plan_launch(plan, alpha, beta, (hipStream_t)stream));
}

static int graph_launch_impl(mfg_grouped_plan* plan, float alpha, float beta, hipStream_t s) {
    if (!plan) return MFG_ERR_INVALID_ARG;
    if (plan->exec && (plan->g_alpha != alpha || plan->g_beta != beta)) {
        MFG_HIP_CHECK(hipGraphExecDestroy(plan->exec));
        MFG_HIP_CHECK(hipGraphDestroy(plan->graph));
        plan->exec = nullptr, plan->graph = nullptr;
    }
    if (!plan->exec) {
        if (!plan->cap_stream) MFG_HIP_CHECK(hipStreamCreateWithFlags(&plan->cap_stream, hipStreamNonBlocking));
        MFG_HIP_CHECK(hipStreamBeginCapture(plan->cap_stream, hipStreamCaptureModeThreadLocal));
        int st = plan_launch(plan, alpha, beta, plan->cap_stream);
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(plan->cap_stream, &g);
        if (st != MFG_OK) {
            if (g) (void)hipGraphDestroy(g);
            return st;
        }
        if (e != hipSuccess) return hip_fail(e);
        hipGraphExec_t x = nullptr;
        e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(g);
            return hip_fail(e);
        }
        plan->graph = g, plan->exec = x, plan->g_alpha = alpha, plan->g_beta = beta;
    }
    MFG_HIP_CHECK(hipGraphLaunch(plan->exec, s));
    return MFG_OK;
}

extern "C" int mfg_grouped_graph_launch(mfg_grouped_plan* plan, float alpha, float beta, void* stream) {
    MFG_GUARD(graph_launch_impl(plan, alpha, beta, (hipStream_t)stream));
}

extern "C" int mfg_grouped_plan_info(const mfg_grouped_plan* plan, double* flops, double* bytes,
                                     int64_t* work_items) {
    if (!plan) return MFG_ERR_INVALID_ARG;
    if (flops) *flops = plan->flops;
    if (bytes) *bytes = plan->bytes;
    if (work_items) *work_items = plan->nwork;
    return MFG_OK;
}

extern "C" int mfg_grouped_plan_destroy(mfg_grouped_plan* plan) {
    if (!plan) return MFG_ERR_INVALID_ARG;
    plan_free(plan);
    return MFG_OK;
}

// ----------------------------------------------------------------- converts
extern "C" int mfg_round_f16(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* out, int64_t ldo,
                             void* stream) {
    int st = validate_matrix(rows, cols, X, ldx);
    if (st == MFG_OK) st = validate_matrix(rows, cols, out, ldo);
    if (st != MFG_OK) return st;
    MFG_GUARD(launch_round_f16(rows, cols, X, ldx, static_cast<uint16_t*>(out), ldo, (hipStream_t)stream));
}

extern "C" int mfg_round_bf16(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* out, int64_t ldo,
                              void* stream) {
    int st = validate_matrix(rows, cols, X, ldx);
    if (st == MFG_OK) st = validate_matrix(rows, cols, out, ldo);
    if (st != MFG_OK) return st;
    MFG_GUARD(launch_round_bf16(rows, cols, X, ldx, static_cast<uint16_t*>(out), ldo, (hipStream_t)stream));
}

extern "C" int mfg_split_f16(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* head, void* resid,
                             int64_t ldo, double* norms, void* stream) {
    int st = validate_matrix(rows, cols, X, ldx);
    if (st == MFG_OK) st = validate_matrix(rows, cols, head, ldo);
    if (st == MFG_OK) st = validate_matrix(rows, cols, resid, ldo);
    if (st != MFG_OK) return st;
    MFG_GUARD(launch_split_f16(rows, cols, X, ldx, static_cast<uint16_t*>(head), static_cast<uint16_t*>(resid), ldo,
                               norms, (hipStream_t)stream));
}

extern "C" int mfg_quantize_fp8(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* codes, int64_t ldo,
                                float* scales, void* stream) {
    int st = validate_matrix(rows, cols, X, ldx);
    if (st == MFG_OK) st = validate_matrix(rows, cols, codes, ldo);
    if (st != MFG_OK) return st;
    if (rows > 0 && cols > 0 && !scales) return MFG_ERR_INVALID_ARG;
    MFG_GUARD(launch_quantize_fp8(rows, cols, X, ldx, static_cast<uint8_t*>(codes), ldo, scales, (hipStream_t)stream));
}

static int convert_impl(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* out, int64_t ldo, int mode,
                        hipStream_t s) {
    int st = validate_matrix(rows, cols, X, ldx);
    if (st == MFG_OK) st = validate_matrix(rows, cols, out, ldo);
    if (st != MFG_OK) return st;
    const int m = mode & MFG_MODE_MASK;
    uint16_t* o16 = static_cast<uint16_t*>(out);
    switch (m) {
        case MFG_F32:
            if (rows == 0 || cols == 0) return MFG_OK;
            MFG_HIP_CHECK(hipMemcpy2DAsync(out, (size_t)ldo * 4, X, (size_t)ldx * 4, (size_t)cols * 4, (size_t)rows,
                                           hipMemcpyDeviceToDevice, s));
            return MFG_OK;
        case MFG_F16: return launch_round_f16(rows, cols, X, ldx, o16, ldo, s);
        case MFG_BF16: return launch_round_bf16(rows, cols, X, ldx, o16, ldo, s);
        case MFG_F16_REFINE_A:
        case MFG_F16_SPLIT3:
        case MFG_F16_SPLIT4: return launch_split_f16(rows, cols, X, ldx, o16, o16 + rows * ldo, ldo, nullptr, s);
        case MFG_BF16_SPLIT3: return launch_split_bf16(rows, cols, X, ldx, o16, o16 + rows * ldo, ldo, nullptr, s);
        case MFG_FP8_E4M3: {
            uint8_t* c = static_cast<uint8_t*>(out);
            return launch_quantize_fp8(rows, cols, X, ldx, c, ldo,
                                       reinterpret_cast<float*>(c + mfg_fp8_scale_offset(rows, ldo)), s);
        }
        case MFG_BF16_SPLIT6: return MFG_ERR_UNSUPPORTED;  // no preconverted form
        default: return MFG_ERR_INVALID_ARG;
    }
}

extern "C" int mfg_convert(int64_t rows, int64_t cols, const float* X, int64_t ldx, void* out, int64_t ldo, int mode,
                           void* stream) {
    MFG_GUARD(convert_impl(rows, cols, X, ldx, out, ldo, mode, (hipStream_t)stream));
}

extern "C" int mfg_error_norms(int64_t M, int64_t N, const float* C, int64_t ldc, const double* Cref, int64_t ldr,
                               double* out4, void* stream) {
    int st = validate_matrix(M, N, C, ldc);
    if (st == MFG_OK) st = validate_matrix(M, N, Cref, ldr);
    if (st != MFG_OK) return st;
    if (!out4) return MFG_ERR_INVALID_ARG;
    MFG_GUARD(launch_error_norms(M, N, C, ldc, Cref, ldr, out4, (hipStream_t)stream));
}

// ------------------------------------------------------------------ autotune
static int autotune_impl(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                         float* C, int64_t ldc, int mode, int reps, int* best_config, float* best_ms, hipStream_t s) {
    int st = validate_gemm(M, N, K, A, lda, B, ldb, C, ldc, mode);
    if (st != MFG_OK) return st;
    if (reps < 1 || M == 0 || N == 0) return MFG_ERR_INVALID_ARG;
    const int m = mode & MFG_MODE_MASK;
    const int ncfg = mfg_num_configs(m);
    if (ncfg <= 0) return MFG_ERR_INVALID_ARG;
    std::vector<char> timed((size_t)ncfg, 0);
    float* ref = nullptr;
    unsigned long long* cnt = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int best = 0;
    float bms = 0.f;
    auto cleanup = [&]() {
        if (ref) (void)hipFree(ref);
        if (cnt) (void)hipFree(cnt);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    if (hipMalloc(&ref, (size_t)M * N * sizeof(float)) != hipSuccess ||
        hipMalloc(&cnt, sizeof(unsigned long long)) != hipSuccess) {
        cleanup();
        return MFG_ERR_NO_MEMORY;
    }
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        cleanup();
        return MFG_ERR_HIP;
    }
    // beta = 0: C is output only, so every run starts from the same state.
    st = gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, 1.f, 0.f, mode, 0, s);
    if (st == MFG_OK &&
        hipMemcpy2DAsync(ref, (size_t)N * 4, C, (size_t)ldc * 4, (size_t)N * 4, (size_t)M, hipMemcpyDeviceToDevice,
                         s) != hipSuccess)
        st = MFG_ERR_HIP;
    bms = 3.4e38f;
    // Every configuration the shape takes explicitly, then the default choice
    // where it is none of them: it serves any K and row alignment, and an entry
    // that does not serve a shape leaves that shape to it.
    for (int i = 0; st == MFG_OK && i <= ncfg; ++i) {
        const int c = i < ncfg ? i : kConfigDefault;
        int index = c;
        int r = gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, 1.f, 0.f, mode, c, s, nullptr, &index);  // warm-up
        if (r == MFG_ERR_UNSUPPORTED && i < ncfg) continue;
        if (r != MFG_OK) {
            st = r;
            break;
        }
        if (index < 0 || timed[(size_t)index]) continue;
        timed[(size_t)index] = 1;
        float total = 0.f;
        for (int rep = 0; rep < reps && st == MFG_OK; ++rep) {
            if (hipEventRecord(e0, s) != hipSuccess) st = MFG_ERR_HIP;
            r = gemm_impl(M, N, K, A, lda, B, ldb, C, ldc, 1.f, 0.f, mode, c, s);
            if (r != MFG_OK) st = r;
            if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) st = MFG_ERR_HIP;
            float ms = 0.f;
            if (st == MFG_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = MFG_ERR_HIP;
            total += ms;
        }
        if (st != MFG_OK) break;
        if ((st = launch_count_mismatch(M, N, C, ldc, ref, N, cnt, s)) != MFG_OK) break;
        unsigned long long bad = 1;
        if (hipMemcpyAsync(&bad, cnt, sizeof(bad), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            st = MFG_ERR_HIP;
            break;
        }
        const float avg = total / reps;
        if (bad == 0 && avg < bms) bms = avg, best = index;
    }
    cleanup();
    if (st != MFG_OK) return st;
    tuned_store(m, M, N, K, best);
    if (best_config) *best_config = best;
    if (best_ms) *best_ms = bms;
    return MFG_OK;
}

extern "C" int mfg_autotune(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                            float* C, int64_t ldc, int mode, int reps, int* best_config, float* best_ms,
                            void* stream) {
    MFG_GUARD(autotune_impl(M, N, K, A, lda, B, ldb, C, ldc, mode, reps, best_config, best_ms, (hipStream_t)stream));
}
