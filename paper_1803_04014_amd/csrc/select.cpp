// select.cpp -- default tile configuration of each mode when the caller
// asks for none and the tuned table has no entry, from measured sweeps on
// MI355X.  Host code only; kept
// apart from the kernels so that the policy can change without touching
// them.  Configuration indices refer to the menus in gemm16.hip,
// gemm_f8.hip and gemm_f32.hip.
#include <cstdint>

#include <algorithm>

#include "internal.h"

namespace mfg {

// The default of the 16-bit kinds is the candidate with the least estimated
// time: `start` (launch, prologue, one tile's epilogue latency), then per
// tile its part of C at the CU's share of HBM and its 64-deep K stages.  A
// stage costs `lat` us on a workgroup with an otherwise idle chip (latency),
// `full` us per tile when every CU is busy (bandwidth and clock).  Kernels
// that put one workgroup on a CU run ceil(tiles / 256) rounds, with the stage
// between lat and full as the chip fills; the ring kernels share a CU,
// whose n tiles take n full stages but at least one latency.  Figures
// measured on MI355X (random operands): start at 64^3, lat at
// 128 x 128 x 4096, full at 4096^3.  What the choice replaces (the 64 x 64
// tiled kernel served every K % 64 != 0 and every small problem): SPLIT3
// 777 x 1234 x 1999 128 -> 30 us, 4000 x 4000 x 4001 1472 -> 375 us, F16
// 32 x 4096 x 4096 53 -> 18 us, 3000^3 212 -> 71 us, 1024^3 15 -> 7.6 us.
struct Cost16 {
    int cfg, variant;  // menu index; of the ring kernels also launch_ring's variant
    int bm, bn;
    bool shared;       // several workgroups per CU
    float start, lat, full;  // us; us per 64-deep stage
};
static const Cost16 kCostPlain[] = {
    {6, 0, 64, 64, true, 2.6f, 0.27f, 0.19f},       // ring 64 x 64
    {6, 1, 64, 128, true, 2.9f, 0.38f, 0.32f},      // ring 64 x 128
    {28, 0, 128, 128, false, 4.7f, 0.42f, 0.50f},   // q128x128k64s3w2x2g8
    {30, 0, 256, 128, false, 6.9f, 0.68f, 0.83f},   // q256x128k64s3w2x2g8e
    {29, 0, 256, 256, false, 10.0f, 1.20f, 1.44f},  // q256x256k64s2w2x2g8e
};
static const Cost16 kCostRefineA[] = {
    {3, 1, 32, 64, true, 2.9f, 0.36f, 0.20f},
    {3, 0, 64, 64, true, 2.9f, 0.37f, 0.32f},
    {7, 0, 128, 128, false, 5.0f, 0.70f, 0.96f},
    {9, 0, 192, 128, false, 6.4f, 0.93f, 1.26f},
};
static const Cost16 kCostSplit3[] = {
    {3, 1, 32, 64, true, 2.9f, 0.45f, 0.30f},
    {3, 0, 64, 64, true, 2.9f, 0.48f, 0.46f},
    {7, 0, 128, 128, false, 5.0f, 0.95f, 1.30f},
    {9, 0, 192, 128, false, 6.4f, 1.28f, 1.68f},
};
static const Cost16 kCostSplit4[] = {
    {2, 1, 32, 64, true, 2.9f, 0.51f, 0.33f},
    {2, 0, 64, 64, true, 2.9f, 0.53f, 0.53f},
    {5, 0, 128, 128, false, 5.0f, 1.12f, 1.64f},
};

// stages: K stages; ring_cost: factor on the ring kernels' full stages.
static double cost16(const Cost16& c, int64_t M, int64_t N, int64_t stages, int64_t batch, double ring_cost) {
    constexpr double kCus = 256.0, kCBytesPerUs = 20000.0;  // per CU: a 256th of 5.1 TB/s
    const double tiles = (double)cdiv(M, c.bm) * (double)cdiv(N, c.bn) * (double)batch;
    const double load = tiles < kCus ? tiles / kCus : 1.0;
    const double n = tiles <= kCus ? 1.0 : (double)(int64_t)((tiles + kCus - 1.0) / kCus);
    const double ctime = c.bm * c.bn * 4.0 / kCBytesPerUs * load, full = c.full * ring_cost;
    double stage = c.lat + (c.full - c.lat) * load;
    if (c.shared) stage = (n * full > c.lat ? n * full : c.lat) / n;
    return c.start + n * (ctime + (double)stages * stage);
}

static const Cost16& least_cost(const Cost16* c, int n, int64_t M, int64_t N, int64_t stages, int64_t batch,
                                double ring_cost, bool ring_only) {
    int best = 0;
    double least = cost16(c[0], M, N, stages, batch, ring_cost);
    for (int i = 1; i < n; ++i) {
        if (ring_only && !c[i].shared) continue;
        const double t = cost16(c[i], M, N, stages, batch, ring_cost);
        if (t < least) least = t, best = i;
    }
    return c[best];
}

static const Cost16& pick16(int kind, int64_t M, int64_t N, int64_t K, int64_t batch, bool ring_only) {
    const Cost16* c = kCostSplit3;
    int n = (int)(sizeof(kCostSplit3) / sizeof(Cost16));
    if (kind == K_F16 || kind == K_BF16) c = kCostPlain, n = (int)(sizeof(kCostPlain) / sizeof(Cost16));
    else if (kind == K_REFINE_A) c = kCostRefineA, n = (int)(sizeof(kCostRefineA) / sizeof(Cost16));
    else if (kind == K_SPLIT4) c = kCostSplit4, n = (int)(sizeof(kCostSplit4) / sizeof(Cost16));
    // rows of K % 64 != 0 are not whole 128-byte lines: the small tiles draw up
    // to a fifth more of them (SPLIT4 3000^3: 0.69 us per stage, 4096^3: 0.55)
    return least_cost(c, n, M, N, cdiv(K, 64), batch, K % 64 != 0 ? 1.2 : 1.0, ring_only);
}

// Whether the simple kernel (one wavefront per 32 x 32 block, no LDS) beats the
// ring kernels: a short K, or many thin problems that would leave most of the
// ring's tiles empty.  As in pick_config_f32, both are estimated in us as the
// latency of one block or tile, or their sum (ns each) once the chip is full.
// Fitted per kind on shapes where both were timed (410 F16, 180 to 208 each of
// the others: batches of thin problems, single ones up to K = 400): 0.2% to
// 0.9% slower on average than the better of the two, the ring alone 9% to 19%.
// F16 136 x 232 x 8 2.6 us simple, 3.0 ring, 4110 of 80 x 16 x 16 9.5 and 22,
// 848 of 328 x 8 x 80 18 and 21; but 304 x 2040 x 24 3.4 and 3.3, 234 of
// 26 x 368 x 80 9.0 and 8.2, 74 of 16 x 136 x 64 3.9 and 3.2.
struct SimpleOrRing {
    double start, per_k;           // simple: latency and its part per K (of 16)
    double block, k, km, kn;       // a block, and per K by how full its rows and columns are
    double shared;                 // factor where blocks of one problem share rows
    double ring_start, ring_stage; // ring: latency and its part per 64-deep stage
    double second;                 // added from two tiles per CU on
    double tile, stage;            // a tile, and its part per stage
};
static bool simple16(int kind, int64_t M, int64_t N, int64_t K, int64_t batch) {
    static const SimpleOrRing plain{2.12, 0.0224, 0.418, 0.0122, 0.0119, 0.0138, 0.89, 2.61, 0.273, 0.51, 1.84, 1.78};
    static const SimpleOrRing refine_a{2.58, 0.025, 0.421, 0.0116, 0.0142, 0.0137, 0.64, 3.69, 0.075, 1.59, 2.59, 1.69};
    static const SimpleOrRing split3{2.43, 0.0395, 0.391, 0.0246, 0.0130, 0.0163, 1.0, 3.36, 0.371, 1.21, 3.92, 2.46};
    static const SimpleOrRing split4{2.62, 0.0385, 0.385, 0.0232, 0.0188, 0.0153, 0.88, 3.42, 0.46, 2.3, 2.84, 3.2};
    const SimpleOrRing& p = kind == K_F16 || kind == K_BF16 ? plain
                            : kind == K_REFINE_A            ? refine_a
                            : kind == K_SPLIT4              ? split4
                                                            : split3;
    const double mb = (double)cdiv(M, 32), nb = (double)cdiv(N, 32), fm = (double)M / (32.0 * mb), fn = (double)N / (32.0 * nb);
    const double blocks = mb * nb * (double)batch, tiles = (double)(cdiv(M, 64) * cdiv(N, 64)) * (double)batch;
    const double k16 = (double)(cdiv(K, 16) * 16), stages = (double)cdiv(K, 64);
    const double per_block = (p.block + k16 * (p.k + p.km * fm + p.kn * fn)) * (batch == 1 ? p.shared : 1.0);
    const double latency = p.ring_start + p.ring_stage * stages + (tiles > 256.0 ? p.second : 0.0);
    return std::max(p.start + p.per_k * k16, 1.7 + blocks * per_block * 1e-3) <=
           std::max(latency, 1.7 + tiles * (p.tile + p.stage * stages) * 1e-3);
}

// Index 0, the simple kernel, also where rows are not 16-byte aligned.
int pick_config16(int kind, int64_t M, int64_t N, int64_t K, bool vec_ok, int64_t batch) {
    if (!vec_ok || simple16(kind, M, N, K, batch)) return 0;
    return pick16(kind, M, N, K, batch, false).cfg;
}

int pick_ring16(int kind, int64_t M, int64_t N, int64_t K, int64_t batch) {
    return pick16(kind, M, N, K, batch, true).variant;
}

// FP8: as for the 16-bit kinds, per 128-deep stage (start at 64 x 64 x 128,
// lat at 128 x 128 x 4096, full at 4096^3).  The simple kernel is left with
// rows of A that are not 16-byte aligned.
static const Cost16 kCostF8[] = {
    {2, 0, 64, 64, true, 2.4f, 0.27f, 0.195f},
    {2, 1, 64, 128, true, 2.9f, 0.33f, 0.268f},
    {2, 2, 128, 128, true, 3.6f, 0.55f, 0.41f},
    {3, 0, 256, 128, false, 6.4f, 0.69f, 0.755f},
    {4, 0, 256, 256, false, 9.6f, 1.10f, 1.12f},
};
static const Cost16& pick8(int64_t M, int64_t N, int64_t K, bool ring_only) {
    return least_cost(kCostF8, (int)(sizeof(kCostF8) / sizeof(Cost16)), M, N, cdiv(K, 128), 1, 1.0, ring_only);
}

// B as row-major codes: the tiled kernels need a launch that transposes it
// first, the simple kernel reads it as it is, and is the faster one for a short
// K.  us of a call, the GPU kept busy by the ones before: the simple kernel's
// is its 64-deep steps' latency (a step of whole 32-byte pieces of A is half as
// long) or, with many 32 x 32 blocks, their sum; the other two launches take
// 6.8 at least.  64 x 64 x 64 3.8 us against 6.6, 896 x 128 x 64 3.8 and 6.8,
// 64 x 160 x 100 5.9 and 7.5; but 64 x 128 x 256 8.3 and 6.6, 2336 x 5664 x 128
// 28 and 17 (of 250 random shapes up to K = 420 the choice costs 0.2% on
// average; the tiled kernels alone 25%).
static bool simple_f8(int64_t M, int64_t N, int64_t K) {
    const double steps = (double)cdiv(K, 64), blocks = (double)(cdiv(M, 32) * cdiv(N, 32));
    const double tiles = (double)(cdiv(M, 64) * cdiv(N, 64));
    double simple, tiled;
    if (M % 32 == 0 && K % 64 == 0) simple = std::max(2.35 + 1.45 * steps, 3.3 + blocks * (0.6 + 0.7 * steps) * 1e-3);
    else if (M % 32 == 0 && K % 32 == 0) simple = std::max(3.3 + 1.55 * steps, 3.5 + blocks * (0.5 + 1.1 * steps) * 1e-3);
    else simple = std::max(2.4 + 2.5 * steps, 3.5 + blocks * (0.9 + 1.2 * steps) * 1e-3);
    if (K % 128 == 0) tiled = std::max(6.8, 5.0 + tiles * 3.5e-3);
    else tiled = (N <= 32 ? 6.8 : 7.5) + tiles * 3.4e-3;
    return simple <= tiled;
}

int pick_config_f8(int64_t M, int64_t N, int64_t K, bool vec_ok, bool codes) {
    if (!vec_ok || M < 1 || N < 1 || K < 1 || (codes && simple_f8(M, N, K))) return 0;
    return pick8(M, N, K, codes && K % 128 != 0).cfg;
}

int pick_ring_f8(int64_t M, int64_t N, int64_t K) { return pick8(M, N, K, true).variant; }

// FP32: the simple kernel (one wavefront per 32 x 32 block, no LDS) where K is
// short, or where many thin problems would leave most of the ring's 64 x 64
// tiles empty; else the ring.  Both estimated in us as the latency of one block
// or tile, or their sum once the chip is full: a block takes less the emptier
// it is (fewer of its loads are in range) and where it shares rows with others
// of its problem, a tile of the ring does not.  vec: the ring loads 16-byte
// pieces (aligned rows, K % 4 == 0).
// Fitted on 999 shapes where both were timed (batches of thin ones, single ones
// up to K = 200): 0.3% slower on average than the better of the two, where the
// ring alone is 15%.  1055 x 18 x 4 2.7 us simple, 4.2 ring, 543 x 17 x 24 3.5
// and 4.2, 411 of 8 x 376 x 16 7.2 and 13.3, 1130 of 14 x 591 x 96 110 and 146;
// but 3241 x 2652 x 28 17 and 14, 34 of 360 x 32 x 152 9.7 and 6.3, 1903 of
// 126 x 39 x 209 279 and 98.
int pick_config_f32(int64_t M, int64_t N, int64_t K, bool vec, int64_t batch) {
    const double mb = (double)cdiv(M, 32), nb = (double)cdiv(N, 32), fm = (double)M / (32.0 * mb), fn = (double)N / (32.0 * nb);
    const double blocks = mb * nb * (double)batch, tiles = (double)(cdiv(M, 64) * cdiv(N, 64)) * (double)batch;
    const double k8 = (double)(cdiv(K, 8) * 8), k32 = (double)(cdiv(K, 32) * 32);
    const double per_k = (vec ? 0.0171 + 0.0252 * fm + 0.0193 * fn : 0.0270 + 0.0313 * fm + 0.0067 * fn) * (batch == 1 ? 0.71 : 1.0);
    const double simple = std::max(1.83 + (vec ? 0.060 : 0.053) * k8, 2.0 + blocks * per_k * k8 * 1e-3);
    const double latency = (vec ? 2.93 + 0.0207 * k32 : 3.43 + 0.0235 * k32) * (tiles > 256.0 ? 1.4 : 1.0);
    const double per_tile = (K <= 64 ? 2.9 : 5.8) + (vec ? 0.0603 : 0.0714) * k32;
    return simple <= std::max(latency, 2.0 + tiles * per_tile * 1e-3) ? 0 : 1;
}

// The ring tile with the least estimated time: a start-up, then per round of
// 256 tiles the tile's part of C and its 32-deep stages.  All are bound by
// the matrix cores, so tiles sharing a CU take their times one after the
// other; the larger ones spend a little less per flop, the smaller ones
// waste less of the last round.  us per stage measured at 4096^3 (latency
// included: at 128 x 128 x 4096 it is 0.63 / 1.12 / 2.08).
int pick_ring_f32(int64_t M, int64_t N, int64_t K, int64_t batch, bool vec) {
    struct {
        int bm, bn;
        double vec_us, any_us;
    } const tile[] = {{64, 64, 0.545, 0.75}, {64, 128, 1.043, 0.0}, {128, 128, 2.086, 2.63}};
    int best = 0;
    double least = 0.0;
    for (int i = 0; i < 3; ++i) {
        const double us = vec ? tile[i].vec_us : tile[i].any_us;
        if (us == 0.0) continue;
        const double tiles = (double)cdiv(M, tile[i].bm) * (double)cdiv(N, tile[i].bn) * (double)batch;
        const double t = (double)(int64_t)((tiles + 255.0) / 256.0) *
                         (tile[i].bm * tile[i].bn * 4.0 / 20000.0 + (double)cdiv(K, 32) * us);
        if (i == 0 || t < least) least = t, best = i;
    }
    return best;
}

}  // namespace mfg
