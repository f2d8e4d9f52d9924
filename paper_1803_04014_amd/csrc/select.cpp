// select.cpp -- default tile configuration of each mode when the caller
// asks for none and the tuned table has no entry, from measured sweeps on
// MI355X.  Host code only; kept
// apart from the kernels so that the policy can change without touching
// them.  Configuration indices refer to the menus in gemm16.hip,
// gemm_f8.hip and gemm_f32.hip.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.h"

namespace mfg {

// The default of the 16-bit kinds and of FP8 is the candidate with the least
// estimated time.  A kernel that puts one workgroup on a CU runs its tiles in
// rounds of 256: `start` once, per round the tile's part of C at the CU's share
// of HBM and its K stages, and `tile` between rounds (prologue and epilogue).
// A stage of one round takes `lat`, the latency of its loads, and up to `grow`
// more as the chip fills; of further rounds `full`, bandwidth and clock, of a
// last one that fills part of the chip the most of the way back to the former.  The
// ring kernels share a CU: its tiles take their parts of C, `tile` and `full`
// stages one after the other, but no less than one latency.  Where K is not a
// multiple of 64 a stage takes `rag` and `rag_full` times that: the pipelined
// kernels choose an address for every load, and rows are not whole lines.
// us, fitted per kind on 200 to 660 shapes with every candidate timed (64 to
// 16384 x 64 to 280000 x 64 to 16000, random operands): 0.0% to 0.3% slower on
// average than the best candidate, 0.1% to 0.9% where K % 64 != 0, FP8 0.7%.  A
// first fit, whose latencies did not grow with the load and whose rounds cost no
// more than their stages, lost 0.2% to 2.1% and 0.8% to 3.7% (BF16 1792 x 832 x
// 10368 66 us on the ring, 60 on 128 x 128; F16 2752 x 42432 x 128 158 on 128 x
// 128, 123 on 256 x 256; SPLIT4 12480 x 832 x 448 48.9 on 128 x 128, 44.4 on the
// ring; FP8 1472 x 4096 x 2304 1.16 times 256 x 128).  What the choice replaced (a
// 64 x 64 tiled kernel served every K % 64 != 0 and every small problem): SPLIT3
// 777 x 1234 x 1999 128 -> 30 us, 4000 x 4000 x 4001 1472 -> 375, F16 32 x 4096
// x 4096 53 -> 18, 3000^3 212 -> 71, 1024^3 15 -> 7.6.
struct Cost {
    int cfg, variant;  // menu index; of the ring kernels also their variant
    int bm, bn;
    bool shared;       // several workgroups per CU
    float start, lat, grow, full, tile, rag, rag_full;
};
static const Cost kCostPlain[] = {
    {6, 0, 64, 64, true, 2.91f, 0.235f, 0.033f, 0.182f, 0.057f, 1.00f, 1.20f},     // ring 64 x 64
    {6, 1, 64, 128, true, 3.27f, 0.370f, 0.062f, 0.298f, 0.035f, 0.95f, 1.08f},    // ring 64 x 128
    {28, 0, 128, 128, false, 4.37f, 0.326f, 0.137f, 0.485f, 1.26f, 1.35f, 1.06f},  // q128x128k64s3w2x2g8
    {30, 0, 256, 128, false, 5.75f, 0.589f, 0.178f, 0.768f, 1.16f, 1.20f, 1.09f},  // q256x128k64s3w2x2g8e
    {29, 0, 256, 256, false, 6.79f, 1.060f, 0.383f, 1.260f, 1.61f, 1.13f, 1.04f},  // q256x256k64s2w2x2g8e
};
static const Cost kCostRefineA[] = {
    {3, 0, 64, 64, true, 2.76f, 0.358f, 0.018f, 0.282f, 0.024f, 1.08f, 1.01f},
    {3, 1, 32, 64, true, 2.79f, 0.316f, 0.022f, 0.187f, 0.029f, 1.08f, 1.22f},
    {7, 0, 128, 128, false, 3.94f, 0.697f, 0.160f, 0.962f, 0.70f, 1.02f, 1.00f},
    {9, 0, 192, 128, false, 5.42f, 0.816f, 0.283f, 1.290f, 2.24f, 1.08f, 1.05f},
};
static const Cost kCostSplit3[] = {
    {3, 0, 64, 64, true, 3.04f, 0.444f, 0.011f, 0.425f, 0.035f, 1.08f, 1.10f},
    {3, 1, 32, 64, true, 2.86f, 0.411f, 0.020f, 0.297f, 0.254f, 1.08f, 1.08f},
    {7, 0, 128, 128, false, 4.38f, 0.898f, 0.359f, 1.140f, 1.77f, 1.06f, 1.11f},
    {9, 0, 192, 128, false, 5.77f, 1.130f, 0.454f, 1.540f, 2.98f, 1.08f, 1.05f},
};
static const Cost kCostSplit4[] = {
    {2, 0, 64, 64, true, 2.98f, 0.523f, 0.025f, 0.485f, 0.035f, 1.05f, 1.06f},
    {2, 1, 32, 64, true, 2.65f, 0.475f, 0.023f, 0.331f, 0.469f, 1.06f, 1.15f},
    {5, 0, 128, 128, false, 4.30f, 0.965f, 0.455f, 1.300f, 2.41f, 1.17f, 1.15f},
};

// What a problem adds to the candidates' figures: factors on the ring kernels'
// full stages, on their part of C and on their whole time, and whether K is
// whole stages.
struct ProblemCost {
    double stage = 1.0, c = 1.0, ring = 1.0;
    bool ragged = false;
};

static double cost_of(const Cost& c, int64_t M, int64_t N, int64_t stages, int64_t batch, const ProblemCost& add) {
    constexpr double kCus = 256.0, kCBytesPerUs = 20000.0;  // per CU: a 256th of 5.1 TB/s
    const double rounds = (double)cdiv(M, c.bm) * (double)cdiv(N, c.bn) * (double)batch / kCus;
    const double load = rounds < 1.0 ? rounds : 1.0, ctime = c.bm * c.bn * 4.0 / kCBytesPerUs;
    const double first = (c.lat + c.grow * load * load) * (add.ragged ? c.rag : 1.0), k = (double)stages;
    const double each = c.full * (add.ragged ? c.rag_full : 1.0);
    // rounds that are run (a fraction of many: their ends drift apart)
    const double n = rounds <= 1.0 ? 1.0 : rounds <= 4.0 ? std::ceil(rounds) : rounds + 0.5;
    if (c.shared) {
        const double full = std::ceil(rounds) * each * add.stage;
        return add.ring * (c.start + (ctime + c.tile) * rounds * add.c + k * (n == 1.0 || full < first ? first : full));
    }
    double sum = n * each;
    if (n == 1.0) sum = first;
    else if (rounds < n) {
        const double part = rounds - (n - 1.0), last = (c.lat + c.grow * part * part) * (add.ragged ? c.rag : 1.0);
        if (last < each) sum -= 0.8 * (each - last);
    }
    return c.start + (n - 1.0) * c.tile + n * ctime * load + k * sum;
}

static const Cost& least_cost(const Cost* c, int n, int64_t M, int64_t N, int64_t stages, int64_t batch,
                              const ProblemCost& add, bool ring_only) {
    int best = 0;
    double least = cost_of(c[0], M, N, stages, batch, add);
    for (int i = 1; i < n; ++i) {
        if (ring_only && !c[i].shared) continue;
        const double t = cost_of(c[i], M, N, stages, batch, add);
        if (t < least) least = t, best = i;
    }
    return c[best];
}

static const Cost& pick16(int kind, int64_t M, int64_t N, int64_t K, int64_t batch, bool ring_only) {
    const Cost* c = kCostSplit3;
    int n = (int)(sizeof(kCostSplit3) / sizeof(Cost));
    const bool plain = kind == K_F16 || kind == K_BF16;
    if (plain) c = kCostPlain, n = (int)(sizeof(kCostPlain) / sizeof(Cost));
    else if (kind == K_REFINE_A) c = kCostRefineA, n = (int)(sizeof(kCostRefineA) / sizeof(Cost));
    else if (kind == K_SPLIT4) c = kCostSplit4, n = (int)(sizeof(kCostSplit4) / sizeof(Cost));
    ProblemCost add;
    add.ragged = K % 64 != 0;
    // past the 256 MB of the last cache the small tiles' repeated reads come from
    // HBM (F16 320 x 18176 x 13952: 0.40 us per stage, 0.31 below), and so do,
    // beside a plain kind's few stages, the writes of C (1344 x 83200 x 192: 185 us
    // against 148 on 256 x 256)
    const double planes_a = plain ? 1.0 : 2.0, planes_b = plain || kind == K_REFINE_A ? 1.0 : 2.0;
    const double operands = 2.0 * (double)batch * (double)K * (planes_a * (double)M + planes_b * (double)N);
    if (operands > 256e6) add.stage *= 1.3;
    if (plain && 4.0 * (double)batch * (double)M * (double)N > 256e6) add.c = 1.3;
    // a long K: the pipelined kernels where the two are as good as equal, as the
    // ring's time varies more from shape to shape (F16 1920 x 1024 x 6400, estimated
    // 41.0 and 41.5 us, 46.8 on the ring and 43.1 on 128 x 128)
    if (plain && K >= 24 * 64) add.ring = 1.03;
    return least_cost(c, n, M, N, cdiv(K, 64), batch, add, ring_only);
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

// FP8: per 128-deep stage.  The simple kernel is left with rows of A that are
// not 16-byte aligned.
static const Cost kCostF8[] = {
    {2, 0, 64, 64, true, 2.68f, 0.384f, 0.027f, 0.213f, 0.038f, 1.0f, 1.0f},
    {2, 1, 64, 128, true, 3.05f, 0.302f, 0.017f, 0.364f, 0.044f, 1.0f, 1.0f},
    {2, 2, 128, 128, true, 2.59f, 0.827f, 0.023f, 0.508f, 0.061f, 1.0f, 1.0f},
    {3, 0, 256, 128, false, 5.01f, 0.831f, 0.068f, 0.963f, 1.02f, 1.0f, 1.0f},
    {4, 0, 256, 256, false, 9.00f, 1.040f, 0.021f, 1.210f, 1.27f, 1.0f, 1.0f},
};
static const Cost& pick8(int64_t M, int64_t N, int64_t K, bool ring_only) {
    return least_cost(kCostF8, (int)(sizeof(kCostF8) / sizeof(Cost)), M, N, cdiv(K, 128), 1, ProblemCost{}, ring_only);
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
