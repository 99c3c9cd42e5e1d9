// splitk_plan.hpp -- host-side plan of the split-K launches (which tiles are shared, by how many workgroups, and the
// workspace that takes).  Pure host arithmetic, shared by the C ABI and by the host tests of the workgroup -> tile map.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace coda {

constexpr int64_t PLAN_TILE_M = 256, PLAN_TILE_N = 256;   // the kernels' workgroup tile (checked against the kernel config where both are seen)

// Plan of the shared tiles (tiles and K-steps counted with their ragged edges).  The tiles that would leave compute units
// idle -- all of them when there are fewer than 256, else those of the last, partly filled round of 256 -- form the
// "tail"; its K-steps, laid end to end, are cut into `chunks` equal contiguous ranges, one workgroup each, so that the
// tail takes tail / chunks of a tile time instead of a whole one:
//  * chunks = min(256, tail * parts), parts = min(8, K / 1024): every range gets at least 1024 contraction elements
//    (32 K-steps of 32 bf16, 16 of 64 fp8 elements).  When tail * parts fits the chip every tile is cut into `parts`
//    equal parts; otherwise the 256 ranges straddle tile boundaries (a balanced "stream-K" round);
//  * only when it pays against the exchange of partial tiles through the workspace (256 KB per part, written once and
//    read once: the full-chip exchange costs about 70 us): a workgroup must be spared at least SPLITK_MIN_SPARED_STEPS
//    K-steps of a tile, and must be left with at most SPLITK_MAX_SHARE_NUM / _DEN of one.
// Measured (residual + sum-of-squares program, bf16, against the same launch without workspace): K = 8192: 4 tiles
// 2.7x, 16 tiles 2.4x, 40 tiles +73 %, 64 tiles 1.7x, 72 tiles +18 %, 96 tiles +31 %, 128 tiles +23 %; 272 tiles +36 %,
// 320 tiles +20 %, 384 tiles +10 %, 576 tiles +13 %; K = 4096: 16 tiles +78 %, 64 tiles +21 %, 128 tiles +6 %, 320 tiles
// +8 %, 384 tiles +4 %; K = 2048 (32 K-steps spared at best): 16 tiles +1 to +6 %, 64 tiles -2 %, 384 tiles -9 %.  Rounds
// that are more than half full lose -- 144 tiles -17 %, 160 tiles +0 %, 192 tiles -3 %, 208 tiles -29 % (ranges of 13/16 of
// a tile leave slivers of 1/16, each with its own pipeline fill and exchange), 448 tiles -5 % at K = 8192 and -2 % at
// K = 16384, 496 tiles -19 % -- and run unsplit.  Hence: spared >= 64 K-steps, share <= 1/2 (a round of up to 128 tiles;
// ranges straddle tile boundaries when tail * parts exceeds the chip, e.g. 40 tiles x 8 parts: +73 %).
constexpr int64_t SPLITK_CUS = 256, SPLITK_MAX_PARTS = 8, SPLITK_MIN_K = 1024, SPLITK_MIN_SPARED_STEPS = 64;
constexpr int64_t SPLITK_MAX_SHARE_NUM = 1, SPLITK_MAX_SHARE_DEN = 2;
struct SplitPlan {
    int first;    // tiles below `first` run whole
    int tail;     // number of shared tiles (ids first .. first + tail - 1)
    int chunks;   // workgroups that share them; 0: nothing is shared
    int stride;   // exchange slots per shared tile: the largest number of ranges that reach into one tile
    int pieces;   // 1: every range lies in one tile; 2: ranges straddle tile boundaries (two workgroups per range)
};
// `slots` false: without `stride`, whose count over the tail takes up to a microsecond.
inline SplitPlan plan_splitk(int64_t M, int64_t N, int64_t K, bool f8 = false, bool slots = true)
{
    const SplitPlan none = {0, 0, 0, 0, 1};
    if (M <= 0 || N <= 0 || K <= 0) return none;
    const int64_t tiles = ((M + PLAN_TILE_M - 1) / PLAN_TILE_M) * ((N + PLAN_TILE_N - 1) / PLAN_TILE_N);
    const int64_t scale = f8 ? 2 : 1;                         // an fp8 K-step covers twice the elements in the same time
    const int64_t pairs = (K + scale * 64 - 1) / (scale * 64);   // pairs of K-steps per tile (K-steps of 32 bf16 / 64 fp8 elements)
    int64_t parts = K / (scale * SPLITK_MIN_K);
    if (parts > SPLITK_MAX_PARTS) parts = SPLITK_MAX_PARTS;
    if (parts < 2) return none;
    const int64_t tail = tiles < SPLITK_CUS ? tiles : tiles % SPLITK_CUS;
    if (tail == 0) return none;
    int64_t chunks = tail * parts < SPLITK_CUS ? tail * parts : SPLITK_CUS;
    if (chunks <= tail) return none;
    // K-steps of the longest range against those of a whole tile
    const int64_t longest = 2 * ((tail * pairs + chunks - 1) / chunks);
    if (2 * pairs - longest < SPLITK_MIN_SPARED_STEPS / (f8 ? 2 : 1)) return none;
    if (SPLITK_MAX_SHARE_DEN * tail > SPLITK_MAX_SHARE_NUM * chunks) return none;
    // ranges per tile: tile a is reached by the ranges that hold its first and its last pair, and those in between
    const int64_t total = tail * pairs;
    int64_t stride = 1;
    for (int64_t a = 0; slots && a < tail; ++a) {
        const int64_t c_lo = ((a * pairs + 1) * chunks + total - 1) / total - 1;
        const int64_t c_hi = (((a + 1) * pairs) * chunks + total - 1) / total - 1;
        if (c_hi - c_lo + 1 > stride) stride = c_hi - c_lo + 1;
    }
    return SplitPlan{(int)(tiles - tail), (int)tail, (int)chunks, (int)stride, chunks % tail == 0 ? 1 : 2};
}
constexpr size_t SPLITK_CNT_BYTES = 1024;   // ticket counters (at most 255 shared tiles x 4 bytes), kept apart from the partials
inline size_t splitk_bytes(const SplitPlan &pl)
{
    if (pl.chunks == 0) return 0;
    return SPLITK_CNT_BYTES + (size_t)pl.tail * (size_t)pl.stride * PLAN_TILE_M * PLAN_TILE_N * sizeof(float);
}


// Stages (128 bytes of K, a pair of K-steps) of a plan's longest range.
inline int splitk_longest_stages(const SplitPlan &pl, int64_t K, bool f8)
{
    const int64_t stages = (K * (f8 ? 1 : 2) + 127) / 128;
    return (int)((pl.tail * stages + pl.chunks - 1) / pl.chunks);
}

// The longest chain of additions, in stages, that is no less accurate than a plan's ranges: a tile's stages over the largest number
// of ranges that reach into one.  Ranges that straddle tiles leave most tiles in shorter pieces than the longest range (2 x 16400
// x 23088 against 64 bits: 4.57e-7 shared, 4.72e-7 in chains of the longest range).
inline int splitk_chain(const SplitPlan &pl, int64_t K, bool f8)
{
    const int64_t stages = (K * (f8 ? 1 : 2) + 127) / 128;
    return (int)((stages + pl.stride - 1) / pl.stride);
}

// Plan of the contractions with small output tiles (gemm_small.hpp): bm x bn tiles, each cut along K into `nsplit` ranges
// whose fp32 partials [nsplit][M][N] lie in the workspace.  It takes the place of the shared 256 x 256 tiles where every
// tile of the shape would be shared (plan.first == 0), within the workspace that plan asks for, so that the sizes callers
// see do not depend on which of the two runs.
//
// Up to 64 rows (one tile row) the operands stream from memory once and the small tiles always win: 1 / 32 / 64 rows,
// N x K = 6144 x 4096: 14 / 15 / 17 us against 47; 28672 x 4096: 39 / 41 / 44 against 104; 4096 x 14336: 23 / 25 / 29
// against 75.  One workgroup per CU is the best count there (at 6144 x 4096: 96, 240, 480, 768 workgroups: 18.9, 14.1,
// 15.2, 16.3 us): twice as many pay more exchange and fill for bytes in flight that memory does not need.
//
// Above that, the candidates are modelled in microseconds from their measured parts:
//   one stage (128 bytes of K) of a 128 x 128 tile 0.57, of a 128 x 256 tile 0.83, one workgroup of either per CU
//   partials: written once and read once at 5 TB/s; launches and epilogue: 6
//   one K-step (64 bytes of K) of a 256 x 256 tile 0.83; exchange of its parts 12 and 0.019 per range and slot, 25 more
//   when ranges straddle tiles
// e.g. (128 x 128 / 128 x 256 / 256 x 256, measured; the model is within 6 %, 256 x 256 within 20 %) 509 x 2048 x 8192: 32.5
// / 32.9 / 61.7; 1000 x 2048 x 11264: 64.0 / 58.7 / 90.5; 768 x 4096 x 14336: 137 / 110 / 144; 1024 x 4096 x 14336: 150 / 129 /
// 124, where the large tiles stay.  The small tiles must win by a tenth.  (Two workgroups of 128 x 128 tiles per CU, four
// waves and two stages each, lie between: 384 x 6144 x 4096 40.6, 128 x 256 38.0; 768 x 4096 x 14336 113.)
// Shapes of SMALL_MODEL_TILES tiles of 256 x 256 and more that these figures leave on shared tiles are priced once more: there the small
// tiles fill the chip with one range or two, and the exchange of that many tiles is what costs:
//   launches and epilogue 6; one stage of a 128 x 128 tile 0.57, of a 128 x 256 tile 0.52 and 0.37 more when every CU has one
//   (they share the L2s), 0.05 for a K-contiguous B; partials as above, but not for one range of 128 x 256 tiles, which all
//   programs but RMSNORM_BWD run undivided (that one comes with bf16 A B^T);
//   256 x 256 tiles: a pair of K-steps 1.42; the exchange of parts 4, 0.06 a range, 0.02 a range and slot; where ranges
//   straddle tiles 30, and 1.3, 1.75 or 2 times the longest range, as the pieces of 8, 16 or more ranges repeat.
// Of 110 random shapes that the older figures left on shared tiles those that now take small ones gain 2 to 35 %, 16 % in the mean over
// all: 1232 x 5568 x 15040 329 -> 213 us, 1072 x 3840 x 11072 176 -> 119, 960 x 5376 x 10432 174 -> 127, 1024 x 8192 x 4096 77 -> 62.
// A shape that the first figures give small tiles keeps them, and its tile: back on shared tiles its chains would be up to half as long
// again (fp32 error 12 to 14 % larger) and it would be slower (543 x 8192 x 8192 A B^T 97 us, shared 126; 930 x 6144 x 5632 A B^T 75, 89;
// faster only at few, 1393 x 4088 x 7608 A B^T 148, 109), and the second figures charge partials for one range of 128 x 128 tiles, which
// most programs run undivided (99 x 22016 x 4096 8-bit: 24.2, two ranges of 128 x 256 29.4).
// So does A B^T on shared tiles whose K is no whole number of 128-byte lines: a stage's row of B then lies in two lines, and small tiles
// fetch more rows for what they compute (1128 x 4160 x 12648 with transposed A 195 us, small 233, 768 x 6848 x 7184 8-bit 61, 70; of 150 shapes that
// would move, storing D, the 22 such gain 1 % in the mean, the others 23 %).
// Why from 70 tiles on: of 150 shapes of 70 to 128 that move the plain store gains 23 % in the mean and the RMSNorm backward, which pays for
// its partials in one range as well, 11 % (11 of 128 lose 2 to 8 %, 8-bit and A B, while the other programs of the shape gain 2 to 20 %; the
// plan cannot depend on the program).  At 60 to 69 tiles, below which none would move, 12 of 80 would lose up to 21 % in the plain store and 31
// of 80 in the RMSNorm backward (12 and 2 % faster in the mean): the figures do not hold there.
// Shared tiles stay at 2048 x 4096 x 14336 (179, small 189), 1440 x 4096 x 14336 (164, 181), 384 x 16384 x 14336 A B^T (189, 228).
struct SmallPlan {
    int bm, bn;    // the tile: 32, 64 or 128 rows, 128 (or, with 128 rows, 256) columns
    int nsplit;    // ranges of the contraction; 0: the shape runs on the large tiles
    double us;     // modelled time
    bool fused;    // one range, whose epilogue runs in the same kernel
};
constexpr int64_t SMALL_MODEL_TILES = 70;
constexpr int64_t SMALL_MAX_SPLIT = 16, SMALL_MIN_STAGES = 4;   // beyond that the exchange costs what the ranges save
inline double shared_tiles_us(const SplitPlan &big, int64_t K, bool f8)
{
    const double pairs = splitk_longest_stages(big, K, f8);
    if (big.pieces == 1) return 4.0 + 0.06 * big.chunks + 0.02 * (double)big.chunks * big.stride + 1.42 * pairs;
    int period = big.chunks;                        // ranges after which the pieces of the tiles repeat
    for (int tail = big.tail; tail % 2 == 0 && period % 2 == 0; tail /= 2) period /= 2;
    return 30.0 + 1.42 * pairs * (period <= 8 ? 1.3 : period <= 16 ? 1.75 : 2.0);
}
inline SmallPlan plan_small(int64_t M, int64_t N, int64_t K, bool f8, bool a_k_contiguous, bool b_k_contiguous, const SplitPlan &big)
{
    const SmallPlan none = {0, 0, 0, 0.0, false};
    if (big.chunks == 0 || big.first != 0) return none;
    const int64_t esz = f8 ? 1 : 2, stages = (K * esz + 127) / 128;
    const int64_t budget = (int64_t)splitk_bytes(big) / (M * N * 4);              // ranges whose partials fit
    auto offer = [&](int bm, int bn, double stage_us, double shared_us = 0.0, bool undivided = false) {      // undivided: if in one range
        const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        int64_t ns = SPLITK_CUS / tiles;
        if (ns > SMALL_MAX_SPLIT) ns = SMALL_MAX_SPLIT;
        if (ns > stages / SMALL_MIN_STAGES) ns = stages / SMALL_MIN_STAGES;
        if (ns > budget) ns = budget;
        if (ns < 1) return none;
        const double stage = stage_us + shared_us * (double)(tiles * ns) / (double)SPLITK_CUS;
        return SmallPlan{bm, bn, (int)ns, 6.0 + stage * (double)((stages + ns - 1) / ns) + (undivided && ns == 1 ? 0.0 : (double)(ns * M * N) * 8.0 / 5e6), false};
    };
    if (M <= 64 && a_k_contiguous) return M <= 32 ? offer(32, 128, 0.62) : offer(64, 128, 0.62);
    const SmallPlan narrow = offer(128, 128, 0.57), wide = offer(128, 256, 0.83);
    // one range: most programs run undivided and pay no partials (plan_route), and all take the same plan
    auto cost = [&](const SmallPlan &p) { return p.us - (p.nsplit == 1 ? 0.5 * (double)(M * N) * 8.0 / 5e6 : 0.0); };
    const SmallPlan best = wide.nsplit == 0 || (narrow.nsplit != 0 && cost(narrow) <= cost(wide)) ? narrow : wide;
    const double t_big = 0.83 * 2.0 * splitk_longest_stages(big, K, f8) + 12.0 + 0.019 * big.chunks * big.stride + (big.pieces > 1 ? 25.0 : 0.0);
    if (best.nsplit != 0 && best.us <= 0.9 * t_big) return best;
    if (big.tail < SMALL_MODEL_TILES || (b_k_contiguous && K * esz % 128)) return none;
    const SmallPlan wide2 = offer(128, 256, b_k_contiguous ? 0.57 : 0.52, 0.37, f8 || !b_k_contiguous);
    const SmallPlan best2 = wide2.nsplit == 0 || (narrow.nsplit != 0 && narrow.us <= wide2.us) ? narrow : wide2;
    return best2.nsplit != 0 && best2.us <= 0.95 * shared_tiles_us(big, K, f8) ? best2 : none;
}

// Undivided launches with small tiles, rows x columns of the tile: for what neither plan above divides (a short
// contraction, no workspace) but 256 x 256 tiles leave mostly idle.  Row reductions are per 256 columns (`wide`), A with
// rows not contiguous in K takes 128-row tiles, and the column reduction of RMSNORM_BWD stays on 256-row tiles.
// 128x128_PAIR: two workgroups per CU, so that one's read-modify-write of the gradient runs under the other's contraction.
//
// Model in microseconds: launch, fill and epilogue, then per stage (128 bytes of K) and round of 256 workgroups, as
// measured with cold weights (bf16; before is 256 x 256): 64 x 6144 x 2048: 64x64 15.5, 128x128 20.6, before 45.1; 64 x 22272 x
// 4096: 128x128 41.0, 64x64 50.6, before 83.8, with row sums: 32x256 51.5, 64x256 55.4, before 86.8; 300 x 11008 x 3000 with
// row sums: 64x256 41.1, 128x256 46.0, before 67.8; 509 x 6144 x 2048: 128x128 22.6, 128x256 31.7, before 46.1; 509 x 16384 x
// 2048: 128x256 34.8, 128x128 44.4, before 46.8; 257 x 22312 x 4096: 64x256 105, 128x256 120, 256 x 256 94, which keeps it, as it
// does 1000 x 16384 x 2048 (128x256 66.8, 256 x 256 55.4).
// A plan_small() with one range per tile gives way to these where the model says so, see plan_route; `chains`: those that keep to
// its chain, all but PAIR and 32x256.
// The gradient program also reads and writes 8 bytes per element, of which two workgroups of a CU (PAIR) run a part under each other's contraction.
constexpr int64_t NEVER_STAYS_BYTES = 280ll << 20;    // more than that leaves nothing in the 256 MB Infinity Cache for the next call
enum DirectTile : int { DIRECT_NONE = 0, DIRECT_64x64, DIRECT_32x256, DIRECT_64x256, DIRECT_128x128, DIRECT_128x128_PAIR, DIRECT_128x256 };
enum DirectProgram : int { DIRECT_PROG_LINEAR, DIRECT_PROG_SWIGLU_FWD, DIRECT_PROG_SWIGLU_BWD, DIRECT_PROG_ACCUM, DIRECT_PROG_RMSNORM_BWD };
struct DirectPlan {
    int tile;
    double us;     // modelled time
};
inline DirectPlan plan_direct(int64_t M, int64_t N, int64_t K, bool f8, bool a_k_contiguous, DirectProgram prog, bool wide, const SplitPlan &big_plan,
                              bool chains = false)
{
    DirectPlan best = {DIRECT_NONE, 0.0};
    if (M <= 0 || N <= 0 || K <= 0 || prog == DIRECT_PROG_RMSNORM_BWD) return best;
    // where a workspace lets the last round be shared, the tiles of the whole rounds are the same bits with and without one
    if (big_plan.first > 0) return best;
    const double stages = (double)((K * (f8 ? 1 : 2) + 127) / 128);
    const double rmw = prog == DIRECT_PROG_ACCUM ? (double)M * (double)N * 8.0 / 5e6 : 0.0;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    auto rounds = [&](int64_t t) { return (double)((t + SPLITK_CUS - 1) / SPLITK_CUS); };
    const int64_t big = tiles(PLAN_TILE_M, PLAN_TILE_N);
    const double fill = big < SPLITK_CUS ? (double)big / (double)SPLITK_CUS : 1.0;
    best.us = (prog == DIRECT_PROG_ACCUM ? 0.99 : 0.92) * (6.0 + stages * (1.15 + 0.4 * fill) * rounds(big) + 0.64 * rmw);    // what a small tile has to beat
    const bool gradient = prog == DIRECT_PROG_ACCUM && !f8 && !a_k_contiguous;       // bf16 weight gradients (A^T)
    auto offer = [&](int tile, double us) {
        if (us < best.us) best = DirectPlan{tile, us};
    };
    const bool few = a_k_contiguous && (prog == DIRECT_PROG_LINEAR || prog == DIRECT_PROG_SWIGLU_FWD);
    // weights from HBM: 4.6 TB/s in rows of 64 columns, 5.6 in rows of 128 (28672 x 4096 bf16: 52.9 us, 44.4), 3.9 through one 256-wide
    // workgroup per CU
    auto stream = [&](double us, double rate) {
        const double hbm = (double)N * (double)K * (f8 ? 1.0 : 2.0) / rate;
        return us > hbm ? us : hbm;
    };
    // 8-bit, several rounds of 256-wide tiles: past 16 stages 256 x 256 tiles are ahead by 5 to 20 % (384 x 58320 x 15968: 397,
    // 128x256 486), below that up to as much behind (3598 x 5456 x 352: 45, 37)
    auto crowded = [&](int64_t bm) { return f8 && tiles(bm, 256) > SPLITK_CUS && stages > 16.0; };
    if (few && !wide) offer(DIRECT_64x64, 4.0 + stream(stages * 0.34 * rounds(tiles(64, 64)), 4.6e6));
    if (few && prog == DIRECT_PROG_LINEAR) {
        if (!chains) offer(DIRECT_32x256, 5.3 + stream(stages * 0.55 * rounds(tiles(32, 256)), 3.9e6));
        if (!crowded(64)) offer(DIRECT_64x256, 5.5 + stages * 0.68 * rounds(tiles(64, 256)));
    }
    // every further round pays its fill and epilogue: 897 x 19712 x 200 SwiGLU, five rounds: 28.3, 256 x 256 26.6; 3426 x 2832 x 160
    // 8-bit, three: 17.0, 14.8
    if (!wide) offer(DIRECT_128x128, 2.5 + 2.0 * rounds(tiles(128, 128)) + stream(stages * 0.57 * rounds(tiles(128, 128)), 5.6e6) + rmw);
    // bf16 contractions that 256 x 256 tiles nearly fill one round with: 4096 x 4096 x 32 PAIR 29.2, 256 x 256 27.0; of ten shapes of 200 to 256 tiles,
    // K of 64 to 4000, A^T, PAIR is at most 6 % ahead below 256 and 5 to 40 % behind from 512 on (3584 x 4096 x 64 28.3, 29.0; x 1000 52.3, 49.0)
    const bool bare = !f8 && big <= SPLITK_CUS && fill > 0.8 && (gradient || stages < 4.0);
    // rounds of two per CU; what is left over runs two or one per CU (1424 x 6304 x 12920: 600 tiles lose 30 % to 256 x 256)
    const int64_t pairs = tiles(128, 128), whole = pairs / (2 * SPLITK_CUS), left = pairs % (2 * SPLITK_CUS);
    const double one = left > 0 && left <= SPLITK_CUS ? 1.0 : 0.0, two = (double)whole + (left > SPLITK_CUS ? 1.0 : 0.0);
    const bool paired = prog == DIRECT_PROG_ACCUM && !chains && !bare;
    // up to 256 tiles leave a workgroup without its second: bf16 gradients then take one a CU, in the mean of 102 shapes, K up to 9768, 4 % faster with D
    // cold (9 slower to 29 faster) and 11 % on a D that stays (1000 x 4048 x 504 18.7 -> 17.4, x 816 23.5 -> 20.6; from 257 tiles on 10 to 20 % slower)
    if (paired) offer(gradient && pairs <= SPLITK_CUS ? DIRECT_128x128 : DIRECT_128x128_PAIR, 6.0 + stages * (1.08 * two + 0.66 * one) + 0.55 * rmw);
    if (!crowded(128)) offer(DIRECT_128x256, (6.0 + stages * 0.88 * rounds(tiles(128, 256)) + rmw) * (prog == DIRECT_PROG_ACCUM ? 1.07 : 1.0));
    // bf16 gradients for which that leaves 256 x 256 tiles: both in figures of D moved in rows, cold and by way of the caches, fitted to 555 shapes, K of 16 to
    // 8192 (within 7 %).  They move 147 of the shapes timed, 7 % faster in the mean with D cold (5 slower to 16 faster) and 5 % on a D that stays (14336 x 4096 x
    // 504 140 -> 125, 2048 x 11264 x 2000 126 -> 120), and not 2048 x 16384 x 504 (85.6, PAIR 92.8), 5632 x 2048 x 1000 (42.9, 46.0), 10240 x 5120 x 4096 (398, 438).  D past
    // the caches, which N decides here, stays: 4096 x 28672 x 424 222, PAIR 252.
    if (gradient && paired && best.tile == DIRECT_NONE && (M * N * 4 < NEVER_STAYS_BYTES || N % 32)) {
        const double large = 3.4 + 9.9 * rounds(big) + stages * (1.14 * rounds(big) + 0.25 * (double)big / (double)SPLITK_CUS) + 0.66 * rmw;
        const double pair = 7.6 + stages * (0.91 * two + 0.75 * one) + 0.85 * rmw;
        if (pair < 0.97 * large) best = DirectPlan{DIRECT_128x128_PAIR, pair};
    }
    return best;
}

// 256 x 192 tiles (gemm_kernel_narrow), for undivided bf16 A B without row reductions: the same bits, in another number of rounds.
// One round of 129 to 192 large tiles is one round of three quarters the length: 2560 x 3776 x 512 19.3 -> 15.6 us, 1728 x 5184 x
// 8192 160 -> 136, 2048 x 6144 x 4096 92 -> 82 (the large tiles leave a quarter of the chip idle, so that the rest clocks higher);
// so are two and a bit (7680 x 4608 x 1024, 2.1 rounds in three: 80.7 -> 70.6).  Where the rounds come out alike the large tiles
// are ahead by 3 to 7 % (1728 x 23552 x 4096: 295, 303).  Half a round of them or less stands against one round of 128 x 256 tiles, which
// spread over twice as many compute units: 2996 x 1288 x 7664 108 us, narrow 123, 11518 x 320 x 13128 192, 272; 30 such are 3 to
// 30 % slower, 14 % in the mean.  `direct`: modelled time of the small tiles that the shape would take.
// Model in microseconds, per round: fill and epilogue, then a pair of K-steps, which costs less the fewer of the compute units
// draw power; of 54 shapes on large tiles it takes 28, all of them faster (by 13 % in the mean), and leaves 4 that would gain 2 %.
constexpr int64_t NARROW_TILE_N = 192;
inline bool narrow_is_faster(int64_t M, int64_t N, int64_t K, double direct)
{
    if (M <= 0 || N <= 0 || K <= 0) return false;
    if (((M + PLAN_TILE_M - 1) / PLAN_TILE_M) * ((N + NARROW_TILE_N - 1) / NARROW_TILE_N) <= SPLITK_CUS / 2) return false;
    const double pairs = (double)((K + 63) / 64);
    auto us = [&](int64_t bn, double round, double pair, double idle) {
        const int64_t tiles = ((M + PLAN_TILE_M - 1) / PLAN_TILE_M) * ((N + bn - 1) / bn), rounds = (tiles + SPLITK_CUS - 1) / SPLITK_CUS;
        const double empty = 1.0 - (double)tiles / (double)(rounds * SPLITK_CUS);
        return 3.0 + (double)rounds * (round + pairs * (pair - idle * empty));
    };
    const double narrow = us(NARROW_TILE_N, 6.0, 1.16, 0.5), large = us(PLAN_TILE_N, 8.0, 1.447, 0.7);
    return narrow < 0.97 * (direct < large ? direct : large);
}

// Whether small tiles fetch B past the caches (the non-temporal hint): a weight matrix that one row of tiles reads once, if it will not be
// there when it is read again.  Weights that take their turn through the 256 MB Infinity Cache leave nothing in it for the next pass, and
// bringing them in costs a tenth of the rate.  Whole lines only: of a line that is fetched in two pieces the second must still find it.
// From NEVER_STAYS_BYTES on both sides bear it out: the same matrix again and again gains up to 20 %, with other weights in between 2 to 16 %.
// Under that the hint is a bet that other weights come in between, as in a model of several layers.  What it gains then, and what it
// costs a lone matrix that would have stayed, over some 350 calls on 96 to 258 MiB (microseconds, ordinary -> hint):
//   a workgroup for at least 7/8 of the compute units, up to 32 rows: 2 to 14 % faster; alone 7 % faster to 11 % slower
//     (1 x 28672 x 4096 42.2 -> 38.6, alone 36.3 -> 37.4; 32 x 14336 x 4096 A B^T 26.5 -> 23.9, 22.0 -> 22.9)
//   64 rows in one range: 4 to 14 % faster; 4 % faster to 13 % slower (64 x 28672 x 4096 45.3 -> 43.5, 37.5 -> 42.4)
//   8-bit 128 x 128 tiles, A B^T: 3 to 15 % faster; up to 27 % slower (96 x 28672 x 4096 28.4 -> 25.8, 21.6 -> 26.3)
// Ordinary loads where what is lost alone is not made good: fewer workgroups, whose loads wait longer (2 to 7 %, 8-bit up to 11; 4 to 43 %
// slower alone: 1 x 22016 x 4096 35.6 -> 34.9, 29.7 -> 33.8, 64 x 18432 x 4608 44.5 -> 43.3, 29.9 -> 41.9); 64 rows in several ranges (64 x 14336 x 4096
// 29.1 -> 29.7, 25.2 -> 29.1); 8-bit A B on 128 x 128 tiles (2 to 10 %; up to 38 % slower: 128 x 28672 x 4096 33.4 -> 31.2, 23.2 -> 28.3).  bf16
// at 65 to 128 rows gains nothing in turn either.
constexpr int64_t ONCE_BYTES = 96ll << 20;
inline bool reads_once(int64_t M, int64_t N, int64_t K, bool f8, bool b_k_contiguous, int bm, int ranges, int64_t ldb_bytes, uint64_t b_address)
{
    const int64_t bytes = N * K * (f8 ? 1 : 2), workgroups = (N + 127) / 128 * ranges;
    if (M > bm || ldb_bytes % 128 || b_address % 128 || (bm == 128 && !f8)) return false;
    if (bytes >= NEVER_STAYS_BYTES) return true;
    if (bytes < ONCE_BYTES || workgroups < SPLITK_CUS - SPLITK_CUS / 8) return false;
    return bm == 32 || (bm == 64 ? ranges == 1 : b_k_contiguous);
}

// Whether the gradient program reads and writes D past the caches: where it is too large to stay in them for the next call, from
// NEVER_STAYS_BYTES on.  Whole lines only: of a line in two pieces the caches save the second (2000 x 5208 x 2000 63 us with the hint, without 55).
// Microseconds, ordinary -> hint, one D again and again and two in turn: 4096 x 18432 x 1000 222 -> 216, 231 -> 216; 4096 x 20480 x 512 214 -> 169, 211 -> 202;
// 8192 x 16384 x 1000 416 -> 349, 415 -> 351, x 4096 879 -> 858, 870 -> 885; 8-bit 4096 x 18432 x 1008 171 -> 165, 187 -> 166.
// Below, D may have stayed from the call before, which is worth more than the operands that the hint leaves in the caches.  76 shapes of 33 to 230 MB,
// K of 256 to 3900, one D again and again and as many in turn as 700 MB hold: 256 x 256 tiles 12 % slower in the mean (1 to 28) and 4 % faster (2 % slower to 14
// faster); 128 x 128 two a CU 2 % slower (5 % faster to 8 slower) and 3 % faster (2 % slower to 7 faster).  4096 x 4096 x 256 28 -> 33, 37 -> 33; 2048 x 11264 x
// 1000 65 -> 68, 81 -> 80; 4096 x 11008 x 1000 117 -> 151, 150 -> 151.  On the loads alone the hint costs half of that and gains half.
inline bool gradient_once(int64_t M, int64_t N, int64_t ld_bytes, uint64_t address)
{
    return M * N * 4 >= NEVER_STAYS_BYTES && ld_bytes % 128 == 0 && address % 128 == 0;
}

// Route of a call.  The order of the additions behind an element must not depend on the program, so what divides the
// contraction is decided by the sizes, operand type and layouts alone:
//   whole (of 256 or 192 columns) or undivided small tiles, chain INT32_MAX: the MFMAs of a tile along K from the place that rot_cols says, the same
//     sums on every tile size;
//   shared: the ranges of `shared`;
//   divided: the ranges of `small`, folded every `chain` stages, started at the stage of rot_cols.
// The program chooses only between tiles of one order: an undivided tile takes the place of a division into one range, with
// that range's chain and starting stages (96 x 28672 x 4096 8-bit SwiGLU: 27 us; partials of 11 MB to write, read and run a second
// kernel on are 5 more).  It does not take the place of more ranges, where it would be 5 to 20 % ahead for a program without row reductions (809 x
// 4096 x 4096: 37 us against 44, 512 x 6144 x 4096 A^T B SwiGLU 40, 43) and behind for one with.
// One range of 32- or 64-row tiles needs no partials where the program reduces over no rows (`fused`, gemm_small_stream), all with ordinary
// loads: 1 x 28672 x 4096 bf16 45.0 -> 43.8 us, 32 rows with SwiGLU 45.6 (128 x 128 tiles) -> 43.8, 64 x 32768 x 4096 56.6 -> 50.1, 57 x
// 28672 x 4096 8-bit 32.2 -> 28.5; over 129 to 256 tiles and K of 4096 and 8192 the fastest of all tiles, by 1 to 13 % (one in 76 behind, by 3.5 %).
enum RouteKind : int { ROUTE_WHOLE = 0, ROUTE_SHARED, ROUTE_DIVIDED, ROUTE_DIRECT };
struct Route {
    RouteKind kind;
    int tile;          // ROUTE_DIRECT: a DirectTile
    int chain;         // longest chain of additions in stages; INT32_MAX: one chain (small tiles)
    int rot_cols;      // see SmallParams; ROUTE_WHOLE: GemmParams::rot_cols if positive
    SplitPlan shared;  // ROUTE_SHARED; the workspace that any route asks for
    SmallPlan small;   // ROUTE_DIVIDED
    bool narrow;       // ROUTE_WHOLE: 256 x 192 tiles
};
// Where an undivided tile starts along K if B is K-contiguous.  256 x 256 tiles of a whole bf16 A B^T start by XCD, and small tiles
// with them.  Up to 256 rows (a row of 256 x 256 tiles: no panels to share) the tiles start by column, in steps of 256 (1 x 65536 x 4096
// 97 us, from stage 0 124; 32 x 50256 x 4096 8-bit 40, 54); not where a workspace would leave whole rounds to the 256 x 256 tiles.
constexpr int ROT_XCD = -1;
inline int undivided_rotation(int64_t M, int64_t N, int64_t K, bool f8, bool a_k_contiguous, bool b_k_contiguous, const SplitPlan &big)
{
    if (!b_k_contiguous || K <= 0 || K % (f8 ? 128 : 64)) return 0;
    if (M % PLAN_TILE_M == 0 && N % PLAN_TILE_N == 0) return a_k_contiguous && !f8 ? ROT_XCD : 0;
    return M <= PLAN_TILE_M && big.first == 0 ? (int)PLAN_TILE_N : 0;
}
inline Route plan_route(int64_t M, int64_t N, int64_t K, bool f8, bool a_k_contiguous, bool b_k_contiguous, DirectProgram prog, bool wide,
                        bool workspace)
{
    const SplitPlan big = plan_splitk(M, N, K, f8, workspace);      // once a call
    Route r = {ROUTE_WHOLE, DIRECT_NONE, INT32_MAX, undivided_rotation(M, N, K, f8, a_k_contiguous, b_k_contiguous, big), big, {0, 0, 0, 0.0, false}, false};
    DirectPlan direct = plan_direct(M, N, K, f8, a_k_contiguous, prog, wide, big);
    // the contraction is divided only when the caller brought the workspace for it; without one the shape runs undivided
    if (workspace && big.chunks > 0) {
        r.small = plan_small(M, N, K, f8, a_k_contiguous, b_k_contiguous, big);
        if (r.small.nsplit == 0) {
            r.kind = ROUTE_SHARED;
            return r;
        }
        r.chain = splitk_chain(big, K, f8);
        r.rot_cols = (int)PLAN_TILE_N;      // a column of the widest tile
        if (r.small.nsplit == 1) {
            direct = plan_direct(M, N, K, f8, a_k_contiguous, prog, wide, big, true);
            r.small.fused = r.small.bm <= 64 && !wide && (prog == DIRECT_PROG_LINEAR || prog == DIRECT_PROG_SWIGLU_FWD);
        }
        // the figures from SMALL_MODEL_TILES on do not compare with plan_direct's: one range of 128 x 256 tiles runs undivided if it can
        const bool undivided = big.tail >= SMALL_MODEL_TILES && r.small.bn == 256;
        if (r.small.nsplit > 1 || r.small.fused || direct.tile == DIRECT_NONE || (!undivided && r.small.us <= direct.us)) {
            r.kind = ROUTE_DIVIDED;
            return r;
        }
    }
    if (direct.tile != DIRECT_NONE) {
        r.kind = ROUTE_DIRECT;
        r.tile = direct.tile;
    }
    if (r.chain == INT32_MAX && !f8 && a_k_contiguous && !b_k_contiguous && !wide &&
        (prog == DIRECT_PROG_LINEAR || prog == DIRECT_PROG_SWIGLU_FWD) &&
        narrow_is_faster(M, N, K, r.kind == ROUTE_DIRECT ? direct.us : 1e30)) {
        r.kind = ROUTE_WHOLE;
        r.narrow = true;
    }
    return r;
}

}  // namespace coda
