// internal.h -- private declarations shared by libmfgemm's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include <cstddef>
#include <cstdint>

#include "mfgemm.h"

namespace mfg {

// Records a failed HIP call for mfg_last_hip_error() (per thread) and
// returns MFG_ERR_HIP.
int hip_fail(hipError_t e);

#define MFG_HIP_CHECK(call)                                    \
    do {                                                       \
        hipError_t mfg_e_ = (call);                            \
        if (mfg_e_ != hipSuccess) return ::mfg::hip_fail(mfg_e_); \
    } while (0)

// After a kernel launch: report a launch error.
#define MFG_LAUNCH_CHECK() MFG_HIP_CHECK(hipGetLastError())

// Per-(device, stream) workspace.  Returns a device pointer holding at least
// `bytes`, or nullptr with *status set.  The region stays valid until the
// next workspace() call on the same stream; growing it synchronises the
// stream before freeing the old region.
void* workspace(hipStream_t s, size_t bytes, int* status);
// A second, independent per-stream region for reduction partials.
void* partials_ws(hipStream_t s, size_t bytes, int* status);
// Number of compute units of the current device (cached).
int device_cu_count();

// -------------------------------------------------------------- arguments
// One GEMM (or a strided batch of them) on 16-bit planes.  A[p] / B[p] are
// the head (p = 0) and scaled-residual (p = 1) planes.
struct Gemm16Args {
    int64_t M, N, K;
    const uint16_t* A[2];
    const uint16_t* B[2];
    float* C;
    int64_t lda, ldb, ldc;
    int64_t sA, sB, sC;  // batch strides (elements)
    float alpha, beta;
};

struct GemmF32Args {
    int64_t M, N, K;
    const float* A;
    const float* B;
    float* C;
    int64_t lda, ldb, ldc;
    int64_t sA, sB, sC;
    float alpha, beta;
};

struct GemmF8Args {
    int64_t M, N, K;
    const uint8_t* A;    // codes
    const uint8_t* B;
    const uint8_t* Bt;   // B's codes transposed (N x K, ld ldbt), for the tiled kernels
    int64_t ldbt;
    const float* sa;     // ceil(M/128) x ceil(K/128)
    const float* sb;     // ceil(K/128) x ceil(N/128)
    float* C;
    int64_t lda, ldb, ldc;
    float alpha, beta;
};

// Kernel families.  `kind` selects the operand format and products:
// K_BF16_SPLIT3: Eq. 2 without R_A R_B on BF16 head and unscaled BF16 residual planes.
enum Kind16 { K_F16 = 0, K_BF16 = 1, K_REFINE_A = 2, K_SPLIT3 = 3, K_SPLIT4 = 4, K_BF16_SPLIT3 = 5 };

// Tile configurations (index 0 is always the simple one-wave-per-32x32 kernel).
int num_configs16(int kind);
const char* config16_name(int kind, int cfg);
int pick_config16(int kind, int64_t M, int64_t N, int64_t K, bool vec_ok, int64_t batch = 1);
// The tile variant of the ring kernels for a problem (launch_ring's menu).
int pick_ring16(int kind, int64_t M, int64_t N, int64_t K, int64_t batch);
// any_k: cfg came from pick_config16, whose choices serve any K and N; an
// explicit or tuned cfg of the fast and pipelined kernels needs whole stages.
int launch_gemm16(int kind, int cfg, const Gemm16Args& a, int64_t batch, bool vec_ok, hipStream_t s,
                  bool any_k = false);
// Whether a configuration serves a problem (its launch would not return
// MFG_ERR_UNSUPPORTED); a tuned choice that does not is replaced by the
// default.  vec_ok: 16-byte aligned rows of A and B (FP8: of A's codes).
bool config16_ok(int kind, int cfg, int64_t M, int64_t N, int64_t K, int64_t ldc, bool vec_ok);
bool config_f32_ok(int cfg, int64_t ldc, bool vec_ok);

// Refined GEMMs straight from FP32 operands, split while staged (fused.hip).
// Their configurations follow the plane kernels' in a kind's menu.
struct FusedArgs {
    int64_t M, N, K;
    const float* A;
    const float* B;
    float* C;
    int64_t lda, ldb, ldc;
    float alpha, beta;
};
int num_configs_fused(int kind);
const char* config_fused_name(int kind, int cfg);
bool fused_ok(int kind, int cfg, const FusedArgs& a);
int launch_gemm_fused(int kind, int cfg, const FusedArgs& a, hipStream_t s);
bool config_f8_ok(int cfg, int64_t M, int64_t N, int64_t K, int64_t ldc, bool vec_ok);

int num_configs_f32();
const char* config_f32_name(int cfg);
// vec: 16-byte aligned rows and K % 4 == 0.
int pick_config_f32(int64_t M, int64_t N, int64_t K, bool vec, int64_t batch = 1);
// The tile of the ring kernels: 0 64 x 64, 1 64 x 128 (vec only), 2 128 x 128.
int pick_ring_f32(int64_t M, int64_t N, int64_t K, int64_t batch, bool vec);
// any_rows: cfg came from pick_config_f32, whose choices serve any row
// alignment; an explicit or tuned cfg other than 0 needs aligned rows.
int launch_gemm_f32(int cfg, const GemmF32Args& a, int64_t batch, bool vec_ok, hipStream_t s, bool any_rows = false);

int num_configs_f8();
const char* config_f8_name(int cfg);
// vec_ok: 16-byte aligned rows of A's codes; codes: the operands are the
// caller's codes (B to be transposed, K as it is) and not quantised into the
// workspace (B straight into Bt, both zero-filled to whole 128-deep stages).
int pick_config_f8(int64_t M, int64_t N, int64_t K, bool vec_ok, bool codes);
// The ring kernels' tile: 0 64 x 64, 1 64 x 128, 2 128 x 128.
int pick_ring_f8(int64_t M, int64_t N, int64_t K);
// any_k: cfg came from pick_config_f8; an explicit or tuned tiled cfg needs
// K % 128 == 0.
int launch_gemm_f8(int cfg, const GemmF8Args& a, bool vec_ok, hipStream_t s, bool any_k = false);
bool f8_config_needs_bt(int cfg);
// dst (cols x orows) = src^T (rows x cols bytes), zero from row `rows` on.
int launch_transpose_b8(int64_t rows, int64_t orows, int64_t cols, const uint8_t* src, int64_t lds, uint8_t* dst,
                        int64_t ldd, hipStream_t s);

// Conversions (convert.hip).
int launch_round_f16(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* out,
                     int64_t ldo, hipStream_t s);
int launch_round_bf16(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* out,
                      int64_t ldo, hipStream_t s);
int launch_split_f16(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* head,
                     uint16_t* resid, int64_t ldo, double* norms, hipStream_t s);
int launch_split_bf16(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* head,
                      uint16_t* resid, int64_t ldo, double* norms, hipStream_t s);
int launch_split6_bf16(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint16_t* out, int64_t ldo,
                       int64_t kp, bool side_b, hipStream_t s);
int launch_quantize_fp8(int64_t rows, int64_t cols, const float* X, int64_t ldx, uint8_t* codes,
                        int64_t ldo, float* scales, hipStream_t s);
// One FP8 quantisation: codes (ld ldo) of X (rows x cols), transposed if
// `trans` (code of X[r][c] at codes[c * ldo + r]), scales in the tile order of
// X; the codes cover orows x ocols source positions (at least rows x cols,
// within its 128 x 128 tiles), zero beyond the source.
struct QuantJob {
    const float* X;
    uint8_t* codes;
    float* scales;
    int64_t rows, cols, ldx, ldo, orows, ocols;
    int32_t trans;
};
int launch_quantize_fp8_pair(const QuantJob& a, const QuantJob* b, hipStream_t s);
// Conversion jobs: one matrix, rows x cols FP32 at src (ld lds, any
// alignment) into 16-bit library planes at dst (16-byte aligned, ld ldo a
// multiple of 8); kind 0 rne16, 1 rnebf16, 2 FP16 split (head at dst, scaled
// residual at dst + plane, a multiple of 8), 3 BF16 split (unscaled
// residual).  The output is orows x ocols, at least rows x cols, zero beyond
// the source and to the next multiple of 8 columns.
// Job lists (grouped plans over FP32 operands): task = rpt rows of one job
// (one workgroup), about kJobPieces eight-element pieces.
constexpr int kJobPieces = 512;
struct ConvJob {
    const float* src;
    uint16_t* dst;
    int64_t lds, ldo, rows, cols, orows, ocols, plane;
    int32_t kind;
    int32_t rpt;  // rows per task
};
inline int32_t conv_rows_per_task(int64_t rows, int64_t cols) {
    const int64_t cpr = (cols + 7) / 8, r = kJobPieces / (cpr > 0 ? cpr : 1);
    return (int32_t)(r < 1 ? 1 : (r < rows ? r : rows));
}
// Both operands of one GEMM (or of a batch laid out as one tall matrix) in
// one launch; rpt is not used.  MFG_ERR_UNSUPPORTED beyond 2^31 pieces.
int launch_convert_pair(const ConvJob& a, const ConvJob& b, hipStream_t s);
// A (M x K) and B (K x N) in mode m's preconverted storage form at wa, wb
// (library memory, 256-byte aligned, lda_c and ldb_c multiples of 8; FP8: of
// 16); Eq. 1 keeps B's head alone.  capi.cpp.
int convert_operands(int m, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, void* wa, int64_t lda_c,
                     const float* B, int64_t ldb, void* wb, int64_t ldb_c, hipStream_t s);
struct ConvTask {
    int32_t job, row0;
};
int launch_convert_jobs(const ConvJob* jobs, const ConvTask* tasks, int64_t ntasks, hipStream_t s);
int launch_error_norms(int64_t M, int64_t N, const float* C, int64_t ldc, const double* R,
                       int64_t ldr, double* out4, hipStream_t s);
int launch_count_mismatch(int64_t M, int64_t N, const float* C, int64_t ldc, const float* R,
                          int64_t ldr, unsigned long long* out, hipStream_t s);
int launch_scale_c(int64_t M, int64_t N, float* C, int64_t ldc, float beta, int64_t batch,
                   int64_t sC, hipStream_t s);

// Batched and grouped launches (batched.hip).
struct GroupedDesc {  // one problem (host side; the kernel reads GroupedWork)
    int64_t M, N, K, lda, ldb, ldc;
    const uint16_t* A;
    const uint16_t* B;
    float* C;
    int32_t vec;  // 1: 16-byte aligned rows and ld a multiple of 8 (whole 16-byte loads)
    int32_t pad;
    int64_t pa, pb;  // refined kinds: element offsets of the residual planes of A and B (else 0)
};
// Tiled kernels address C with 32-bit buffer offsets within a 32-row block:
// ldc must stay below this bound for them; larger ldc uses the simple
// kernels (single 32 x 32 blocks, 64-bit addressing).
constexpr int64_t kBufferLdcLimit = int64_t(1) << 24;
inline bool buffer_ldc_ok(int64_t ldc) { return ldc < kBufferLdcLimit; }
// The 64-wide pipelined kernels address a tile's operand rows with 32-bit
// byte offsets from its corner (at most 256 rows of A, 64 of B): lda and
// ldb must stay below this bound for the tiled 16-bit kernels; larger ones
// use the simple kernels.
constexpr int64_t kOperandLdLimit = int64_t(1) << 22;
inline bool operand_ld_ok(int64_t lda, int64_t ldb) { return lda < kOperandLdLimit && ldb < kOperandLdLimit; }
// Likewise for the FP8 tiled kernel's code rows (A and transposed B, bytes;
// up to 256 rows per tile).
constexpr int64_t kF8LdLimit = int64_t(1) << 24;

// Output tile classes of the grouped kernel (one workgroup per tile): 128 or
// 64 a side.  Without a tuned entry a problem takes its kind's default.
constexpr int kGroupedTile = 128;        // default for F16, BF16
constexpr int kGroupedTileRefined = 64;  // default for REFINE_A, SPLIT3, SPLIT4, BF16_SPLIT3 (two planes in LDS)
inline int grouped_tile(int kind) { return kind >= K_REFINE_A ? kGroupedTileRefined : kGroupedTile; }
bool grouped_tile_ok(int kind, int tile);
// The classes of a kind, its default first; returns their number (<= 2).
int grouped_tiles(int kind, int* tiles);
// Tuned-table entries of grouped tile classes use mode kGroupedTuneBase + mode
// (config = tile side).
constexpr int kGroupedTuneBase = 32;
// One tile x tile output tile with everything its workgroup
// reads (16 dwords, so that 16 lanes fetch one record with one load each).
struct GroupedWork {
    const uint16_t* A;  // row m0 of the problem's A
    const uint16_t* B;  // column n0 of its B
    float* C;           // element (m0, n0) of its C
    int64_t lda, ldb, ldc;
    int32_t rows, cols;  // of the tile inside the problem: min(tile, M - m0), min(tile, N - n0)
    int32_t K, vec;
};
static_assert(sizeof(GroupedWork) == 64, "a work record is 16 dwords");
int launch_batched_small(int kind, const Gemm16Args& a, int64_t count, bool vec_ok, int num_cu,
                         hipStream_t s);
// Work list of a grouped launch, split into one contiguous range per XCD
// (workgroup b runs on XCD b % kXcds): each problem's tiles stay on one XCD,
// so its operands are fetched into one L2.
constexpr int kXcds = 8;
struct GroupedSplit {
    int64_t off[2][kXcds + 1];  // list 0: aligned rows (vec), ldc < kBufferLdcLimit, lda and ldb < kOperandLdLimit; list 1: the rest
};
// `planes` (if not null) receives two int64 per work item, in work order:
// the problem's residual-plane offsets pa, pb.
// `tile`: the output tile side of the kind that will run the list (grouped_tile);
// `elem`: bytes of an operand element (4: FP32, A and B cast).
void build_grouped_work(const GroupedDesc* descs, int64_t n, std::vector<GroupedWork>& work, GroupedSplit& split,
                        std::vector<int64_t>* planes = nullptr, int tile = kGroupedTile, int elem = 2);
// One launch per non-empty list (the grid of each from grouped_grid) of the
// tile class `tile` (the one the list was built for).  The refined kinds need
// `planes` in device memory, as build_grouped_work wrote it; F16 / BF16
// ignore it (may be null).
// f32: the records' A and B are FP32 matrices (any 4-byte alignment; the
// list's descs carry vec = 1), converted in the kernel; `planes` may be null.
int grouped_launch(int kind, int tile, const GroupedWork* work, const int64_t* planes, const GroupedSplit& split,
                   float alpha, float beta, hipStream_t s, bool f32 = false);
// Workgroups of a list's launch (a multiple of kXcds).
int grouped_grid(const GroupedSplit& split, int list, int kind, int tile);

// Validation (validate.cpp; pure host code).
int validate_gemm(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                  int64_t ldb, const void* C, int64_t ldc, int mode);
int validate_matrix(int64_t rows, int64_t cols, const void* X, int64_t ld);

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace mfg
