// INT8 MFMA GEMM with int32 accumulation and a fused dequantising epilogue (Eq. 9 of the paper) that also
// adds the rank-r LoRA term.  The same kernels serve the forward product (contraction over c_in) and the
// input-gradient product (contraction over c_out).  A is contraction-contiguous; B is either a plain
// contraction-contiguous [N x K] matrix or the packed weight codes (one copy, quaff_internal.h), read as [N x K] by
// the forward product and as [K x N], through transposing LDS reads, by the input-gradient product.
//
//   C[i, j] = row_scale[i] * ( acc1[i, j] * col_scale[j] + acc2[i, j] * col_scale2[j] ) + sum_p T[i, p] L[j, p]
//   acc1 = A B^T   (K long, the hot loop),   acc2 = A2 B2^T   (K2 = padded outlier count, done in the epilogue)
//
// One kernel template (quaff_gemm_dma.h) serves every output that fills the chip: direct-to-LDS operand streaming through a
// ring of stages, v_mfma_i32_32x32x32_i8, XCD-aware tile order; a second one (quaff_gemm_rows.hip) the small ones.  This file
// chooses between them and the tile shape.
#include "quaff_gemm_dma.h"
#include <stdio.h>

namespace quaff {

namespace {
// Shapes a product can take, and the time of each, estimated in us:
//   fixed + round (rounds - 1) + next (n - 1) + chain rounds K / 1000 + 1e-6 (bm + bn) K (unit n + chip load) + n (low + low2)
// with n the tiles of the busiest compute unit (an XCD's region of the tile grid over its 32 units, rounded up), rounds = n / fit
// rounded up, fit the workgroups of the shape that a unit holds together.  (bm + bn) K are the operand bytes of a tile: `unit` is
// their way to one compute unit, `chip` what all units together take of the L2s and the matrix cores' rate (load: tiles / 256, for
// the tiles above 128 x 128 in whole rounds), `chain` the contraction's dependent steps.  low applies with an adapter, low2 on top beyond rank 32 (a second staging round); the shapes of
// quaff_gemm_rows.hip fetch the adapter's operands block by block: low (rank / 16)^2.
// The constants are fitted to 18664 products (1 to 16000 rows, 192 to 16384 columns and contractions, ranks 0 to 64, 0 to 128
// outliers; launch alone, every shape that could be near the best timed, on operands in the caches and on weights that are not), a
// sample of which stands in profiles/gemm_shapes.csv.  The shape chosen takes 1.007 of the time of the best one in the geometric mean
// (at worst 1.58: 601 x 12736 at K = 5632, rank 64, 64 x 128 tiles for 128 x 192), and more than 1.03 of the choice without the
// three tiles of 64 and 128 rows in 1.7 % (forward) and 0.5 % (input gradient) of the products.  With no term for what all
// units fetch together it is 4.1 % and 2.8 % (86 x 1152 at 15360: 16 x 16 for 32 x 32 blocks, 23.9 / 17.9 us; gradient 5723 x
// 6400 at 1280, rank 64: 256 x 256 for 128 x 192 tiles, 128 / 96).
// The three smallest forward shapes are fitted for the choice itself: by how much the time of the chosen one exceeds the best one's, over
// these and 540 more products of up to 1200 rows.  Fitted for their times alone they mixed up neighbours (16 x 9216 at K = 3072: 16 x 16
// for 32 x 64 blocks, forward step at rank 16 22.4 / 20.9; 26 x 3280 at 14896 32 x 32 for 16 x 16, 38.4 / 34.6): more than 1.03 of
// the choice without a term for what all units fetch in 3.9 % of the 540, now 1.7 (342 x 1088 at 896 11.2 / 10.0, 116 x 2880 at 4672, rank 64,
// forward step 34.3 / 31.4).
// What the three tiles give, us, without / with them: 1003 x 2064 at 1040 15.1 / 10.0, 2048 x 1024 at 3072 19.3 / 12.2, 768 x 1536 at
// 1536 13.7 / 7.8, gradient 1003 x 1040 at 2064 with its quantizer 26.0 / 15.3; 0.89 in the geometric mean.
struct Shape { int id, bm, bn, fit; double fixed, round, next, unit, chip, chain, low, low2; };
constexpr Shape kForward[10] = {
    {kTile256x256, 256, 256, 1, 11.09, 8.87, 2.16, 8.78, 11.49, 2.78, 1.34, 8.31},
    {kTile256x288, 256, 288, 1, 11.40, 12.37, 3.01, 8.78, 11.91, 3.42, 1.17, 7.97},
    {kTile256x128, 256, 128, 1, 7.66, 8.24, 1.68, 7.25, 8.38, 2.73, 2.35, 2.92},
    {kTile128x192, 128, 192, 2, 5.66, 1.74, 3.62, 11.03, 4.08, 0.95, 0.91, 2.79},
    {kTile128x128, 128, 128, 1, 5.70, 3.62, 0.99, 7.05, 6.18, 1.08, 0.60, 2.07},
    {kTile64x128, 64, 128, 2, 4.41, 1.84, 1.23, 5.27, 4.82, 1.59, 0.35, 0.65},
    {kTile64x64, 64, 64, 3, 4.29, 1.41, 0.82, 2.27, 6.27, 1.64, 0.24, 0.46},
    {kRows32x64, 32, 64, 4, 4.69, 21.29, 1.20, 3.76, 10.52, 0.60, 0.09, 0.00},
    {kRows32x32, 32, 32, 8, 3.64, 22.94, 0.45, 9.42, 8.02, 0.40, 0.05, 0.00},
    {kRows16x16, 16, 16, 8, 3.35, 3.55, 0.50, 7.34, 11.79, 0.11, 0.02, 0.00}};
constexpr Shape kGradient[9] = {
    {kTile256x256, 256, 256, 1, 10.07, 8.04, 2.10, 8.13, 11.79, 3.11, 1.80, 6.87},
    {kTile256x288, 256, 288, 1, 10.58, 9.94, 2.96, 8.39, 12.99, 3.33, 1.20, 7.43},
    {kTile256x128, 256, 128, 1, 6.51, 5.93, 1.27, 7.90, 8.76, 2.46, 1.29, 4.69},
    {kTile128x192, 128, 192, 2, 3.52, 2.23, 3.02, 11.72, 3.45, 1.03, 0.84, 2.57},
    {kTile128x128, 128, 128, 1, 5.23, 2.21, 1.06, 7.39, 7.89, 0.98, 0.88, 1.67},
    {kTile64x128, 64, 128, 2, 3.84, 0.65, 1.63, 4.85, 5.43, 1.66, 0.34, 0.54},
    {kTile64x64, 64, 64, 3, 3.92, 0.97, 1.13, 1.98, 6.20, 1.86, 0.15, 0.57},
    {kRows32x64, 32, 64, 4, 4.11, 15.67, 2.74, 0.09, 10.34, 1.40, 0.10, 0.00},
    {kRows16x64, 16, 64, 2, 3.93, 8.26, 3.18, 0.14, 14.96, 0.71, 0.08, 0.00}};
// The 128 x 192 tile with at most one tile for every unit takes a ring of three stages (120 KB of LDS: one workgroup per unit) and
// eight wavefronts.  The third stage keeps the operands of the stage after next in flight, which is what a product whose operands
// come from HBM rather than from the Infinity Cache needs (back to back on operand sets that rotate through more than the
// cache holds, two stages / three: o_proj forward 36.2 / 30.5 us, qkv dX 79.2 / 69.8, 8192 -> 3072 forward 74.1 / 61.7; on cached
// operands level).  Eight wavefronts of 32 x 96 against four of 64 x 96: 2048 x 3072 outputs 26.3 / 27.5 us at K = 3072, 55.9 / 57.8 at
// 8192, level at 9216; gradient with its quantizer 34.7 / 36.5, 71.7 / 71.6; 2048 x 2176 at 768 and similar 0.8 of the time.  With more
// tiles than units two workgroups per unit overlap each other's epilogues instead, which needs the smaller ring and four wavefronts
// (4480 x 13376 at 576, rank 64: 115 us, 134 with the deep ring).
constexpr Shape kDeep[2] = {{kTile128x192Deep, 128, 192, 1, 7.22, 3.00, 0.77, 7.15, 7.50, 1.00, 0.83, 2.81},
                            {kTile128x192Deep, 128, 192, 1, 6.87, 2.21, 0.56, 6.59, 6.53, 1.50, 0.89, 1.60}};

double shape_us(const Shape& s, int64_t M, int64_t N, int64_t K, int32_t rank) {
    // (32-bit divisions: M is below 2^30, N below 2^20)
    const uint32_t tm = ((uint32_t)M + s.bm - 1) / (uint32_t)s.bm, tn = ((uint32_t)N + s.bn - 1) / (uint32_t)s.bn;
    const int64_t tiles = (int64_t)tm * tn;
    int64_t n = (tiles + 255) / 256;
    if (n <= 16) {                    // (with many tiles per unit the regions' edges don't matter)
        const TileGrid r = tile_grid((int)tm, (int)tn, s.bm, s.bn);
        n = ((int64_t)r.rm * r.rn + 31) / 32;
    }
    const double more = (double)((n - 1) / s.fit), bytes = 1e-6 * (double)((s.bm + s.bn) * K);
    // (the larger tiles are bound by their rounds, the smaller ones by what they fetch in all)
    const double all = (double)tiles / 256.0, load = s.bm * s.bn <= 128 * 128 ? all : all < 1.0 ? all * (double)n : (double)n;
    const double low = s.id >= kRows16x16 ? s.low * ((rank / 16) * (rank / 16)) : rank > 32 ? s.low + s.low2 : rank > 0 ? s.low : 0.0;
    return s.fixed + s.round * more + s.next * (double)(n - 1) + s.chain * (more + 1.0) * 1e-3 * (double)K +
           bytes * (s.unit * (double)n + s.chip * load) + (double)n * low;
}

int choose_shape(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient, double* us_estimate) {
    int best = -1;
    double best_us = 0.0;
    for (int c = 0; c < (gradient ? 9 : 10); ++c) {
        const Shape* s = gradient ? &kGradient[c] : &kForward[c];
        if (s->id == kTile128x192 && ((M + 127) / 128) * ((N + 191) / 192) <= 256) s = &kDeep[gradient];
        const double us = shape_us(*s, M, N, K, rank);
        if (best < 0 || us < best_us) { best_us = us; best = s->id; }
    }
    *us_estimate = best_us;
    return best;
}

// A second product too wide for the epilogue's LDS staging (more than two 64-wide outlier slices), in a launch with the main product
// or in one of its own that the main product accumulates onto.
// One launch on the tiles that have registers for two sets of accumulators costs the second contraction on top of the first; two
// cost a launch and an output that is written, read (1.5e-7 us a byte) and written again: 2048 x 8192 -> 3072 with 819 outliers
// 74.9 us / 62 in one launch.  Wide outputs keep the two launches, whose products take the 256-row tiles (estimated: 16384 x 5120 ->
// 5120 with 512 outliers 497 us, 540 in one launch), and so do the smallest, by a margin of 5 % (5 x 7424 -> 9408 with 301 outliers
// forward 39.7 / 41.9).
int choose_wide(int64_t M, int64_t N, int64_t K, int64_t K2, int32_t rank) {
    double two, second;
    choose_shape(M, N, K, rank, false, &two);
    choose_shape(M, N, K2, 0, false, &second);
    two += second + 1.5e-7 * 4.0 * (double)M * (double)N;
    int best = -1;
    for (int c = 0; c < 4; ++c) {
        const Shape& s = c == 0 ? kDeep[0] : kForward[3 + c];          // the deep 128 x 192 tile, then 128 x 128, 64 x 128, 64 x 64
        const double us = shape_us(s, M, N, K + (K2 + 127) / 128 * 128, rank);
        if (us * (best < 0 ? 1.05 : 1.0) < two) { two = us; best = s.id; }
    }
    return best;
}
}  // namespace

static hipError_t launch_gemm_one(const GemmArgs& g, bool dump_acc, hipStream_t stream);

// A product whose output is at most 128 tiles of 256 x 192 (a 2048 x 3072 output is exactly 128) with a long
// contraction runs as two workgroups per tile, each over half of the contraction: 30 % fewer operand bytes per
// multiply-add than one 128 x 192 tile per compute unit, whose main loop is bound by the delivery of operands from L2
// into LDS.  The price is one more trip of the output's worth of int32 sums through the L2 (written, read, and
// written back when the kernel ends): measured on 2048 x 3072 outputs, the split loses at K = 3072, breaks even at
// K = 9216 (66.7 against 67.2 us) and wins at K = 16384 (103 against 111 us).
static bool split_applies(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + 255) / 256) * ((N + 191) / 192);
    return K % 256 == 0 && K >= 12288 && tiles > 64 && tiles <= 128;
}
size_t gemm_split_bytes(int64_t M, int64_t N, int64_t K) {
    if (!split_applies(M, N, K)) return 0;
    const size_t tiles = (size_t)((M + 255) / 256) * (size_t)((N + 191) / 192);
    return tiles * 256 + tiles * 512 * 96 * 4;   // two flags per tile in lines of their own, then 96 accumulators of 512 threads
}

// Outputs of at most 128 tiles of 128 x 192 with a long contraction: two or four workgroups per tile share it where that pays for the
// exchange of their sums through the L2.  Estimated as shape_us does, from the same products; 6 % must be gained (of 39 products
// that 2 % would share 16 are faster alone, of these 20 eight).  One workgroup per
// tile in its best shape / two or four, us: forward 763 x 1408 outputs at 14336 37.8 / 33.8 (four), 479 x 2176 at 16384 44.4 / 35.4, 2021 x 1152 at 16384 61.5 / 52.6; input gradient with its quantizer 970 x 2944 <- 16384 83.8 / 78.4.
// Below K = 6144 the tiles of 64 rows are faster (512 x 3072 at 3072 11.7 us, two workgroups per 128 x 192 tile 17.0).
static double shared_us(int parts, int64_t tiles, int64_t K, int32_t rank, bool gradient) {
    struct Parts { double fixed, unit, chip, chain, low, low2; };
    static constexpr Parts kTwo[2] = {{13.53, 7.29, 6.89, 1.48, 1.94, 3.94}, {9.91, 8.60, 7.84, 1.09, 1.47, 5.80}};
    static constexpr Parts kFour[2] = {{11.32, 7.17, 11.02, 1.89, 1.98, 2.77}, {13.51, 8.10, 11.92, 2.12, 2.15, 1.64}};
    const Parts& p = parts == 2 ? kTwo[gradient] : kFour[gradient];
    const double k = (double)K / parts;
    return p.fixed + p.chain * 1e-3 * k + 320e-6 * k * (p.unit + p.chip / 256.0 * (double)(parts * tiles)) + (rank > 0 ? p.low : 0.0) +
           (rank > 32 ? p.low2 : 0.0);
}
// The workgroups of a tile run on one XCD and one of them fills a compute unit: no more of them than the 32 units of an XCD,
// or the last tiles start when the first have ended (1408 x 2112 outputs, 11 x 11 tiles, 18 of them on an XCD, one / two
// workgroups per tile: 27.8 / 40.1 us at K = 4096, 45.1 / 58.1 at 8192; 640 x 2048 outputs, one / four: 25.6 / 30.5 at 4096).
static int small_split(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient, double gain = 1.06) {
    const int64_t tiles = ((M + 127) / 128) * ((N + 191) / 192);
    if (tiles > 128 || K % 256 != 0 || K < 6144) return 1;
    double alone;
    choose_shape(M, N, K, rank, gradient, &alone);
    const double two = gain * shared_us(2, tiles, K, rank, gradient), four = gain * shared_us(4, tiles, K, rank, gradient);
    // (tiles on the busiest XCD: the grid is cut into eight regions of equal size, rounded up)
    const TileMap map = make_tile_map((int)((M + 127) / 128), (int)((N + 191) / 192), 128, 192, 1);
    const int on_xcd = map.rm * map.rn;
    if (4 * on_xcd <= 32 && K % 512 == 0 && four < alone && four < two) return 4;
    return 2 * on_xcd <= 32 && two < alone ? 2 : 1;
}
// Beside the weight gradients of rank 32 and more on a second stream, whose workgroups (88 to 106 KB of LDS) leave no room on a
// compute unit for one of these, some wait for a partner that has no unit yet: 15 % must be gained.  Backward steps with a second
// stream, us, shared / best unshared shape: at rank 64 970 x 2944 <- 16384 147.1 / 139.5, 2021 x 1152 <- 16384 146.5 / 149.2 (expected
// gain 5 to 10 %), at rank 32 1024 x 2048 <- 8192 67.8 / 56.3 (a loss), 768 x 3072 <- 12288 81.0 / 87.5, 479 x 2176 <- 16384 (four) 77.3 / 85.3.
bool gemm_small_split_pays_beside(int64_t M, int64_t N, int64_t K, int32_t rank) { return small_split(M, N, K, rank, true, 1.15) > 1; }
size_t gemm_small_split_bytes(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient) {
    const int parts = small_split(M, N, K, rank, gradient);
    if (parts == 1) return 0;
    const size_t tiles = (size_t)((M + 127) / 128) * (size_t)((N + 191) / 192);
    return tiles * ((size_t)split_flags(parts) * 128 + (size_t)split_slot_sets(parts) * 256 * 96 * 4);
}

bool gemm_takes_rows(int64_t M, int64_t N, int64_t K, int32_t rank) {
    double us;
    return small_split(M, N, K, rank, false) == 1 && choose_shape(M, N, K, rank, false, &us) >= kRows16x16;
}

// A wide second product as a launch of its own, and the product that accumulates onto it.
static GemmArgs second_product(const GemmArgs& g) {
    GemmArgs c{};
    c.A = g.A2; c.lda = g.K2; c.B = g.B2; c.ldb = g.K2;
    c.M = g.M; c.N = g.N; c.K = g.K2;
    c.row_scale = g.row_scale; c.col_scale = g.col_scale2;
    c.C = g.C; c.ldc = g.ldc;
    return c;
}
static GemmArgs main_product(const GemmArgs& g) {
    GemmArgs m = g;
    m.K2 = 0; m.A2 = nullptr; m.B2 = nullptr; m.col_scale2 = nullptr;
    m.accumulate = 1;
    return m;
}

hipError_t launch_gemm(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    ProfScope prof(K_GEMM, stream);
    // (two launches: the first writes row_scale * acc2 * col_scale2, the main product accumulates onto it)
    // bf16 output exists in the single-launch form only
    if (g.C16 && (g.K2 > 128 || dump_acc)) return hipErrorNotSupported;
    if (!dump_acc && g.K2 > 128) {
        const int wide = choose_wide(g.M, g.N, g.K, g.K2, g.r);
        if (wide >= 0) return launch_gemm_wide(g, wide, stream);
        hipError_t e = launch_gemm_one(second_product(g), false, stream);
        if (e != hipSuccess) return e;
        return launch_gemm_one(main_product(g), false, stream);
    }
    return launch_gemm_one(g, dump_acc, stream);
}

// Forward contractions that are 64 more than a multiple of 128: stages of 64 bytes instead of a last stage of 128 that is half
// zeros.  Forward products, us, 64 / 128 bytes: 4096 x 8192 outputs (256 x 256) 27.9 / 29.3 at K = 192, 44.9 / 46.0 at 832, 52.0 / 51.5 at
// 1088, 140.9 / 136.7 at 4160.  The 256 x 128 tile has room for two workgroups on a compute unit with the narrow ring and gains
// at any length: 8192 x 3072 21.9 / 25.4 at 192, 64.8 / 70.3 at 2112, 112.8 / 119.0 at 4160.  Not with outliers on the two largest
// tiles: their epilogue's operands fit side by side in the wide ring only (2423 x 320 -> 5536, rank 16: 23.0 / 17.6; forward step of
// 4712 x 960 -> 15360 at rank 0: 170 / 154).  Not on the narrower tiles: the deep ring of the 128 x 192 tile is ahead (4160 x 896 at 320
// 12.1 / 9.5, 549 x 2624 at 192 11.9 / 9.1) and its two-stage ring level (4800 x 1728 at 320 19.9 / 20.1).
static bool narrow_stages(const GemmArgs& g, int tile) {
    if (g.K % 128 != 64 || tile > kTile256x128) return false;
    return tile == kTile256x128 || (g.K < 1024 && g.K2 == 0);
}

// The shape of one launch.  Which kernel a product with an adapter takes depends on its sizes alone, not on the type of its output and not on the room
// in the workspace: the kernels add the low-rank term in different orders, and a call's last bits may not depend on either.
static int product_tile(const GemmArgs& g, bool dump_acc) {
    const bool gradient = g.b_layout == kPackedKN, one_launch = !dump_acc && !g.accumulate && g.K2 <= 128;
    const int parts = one_launch ? small_split(g.M, g.N, g.K, g.r, gradient) : 1;
    int tile;
    if (g.split_scratch && one_launch && split_applies(g.M, g.N, g.K)) return kTileSplit;
    if (parts > 1 && g.small_split_scratch) return parts == 2 ? kTileSplitSmall2 : kTileSplitSmall4;
    if (parts > 1 && g.r > 0) {
        tile = kTile128x192Deep;         // (no room for the exchange, or not worth it beside a second stream: the shared form's tile and epilogue)
    } else {
        double us;
        tile = choose_shape(g.M, g.N, g.K, g.r, gradient, &us);
    }
    if (!gradient && narrow_stages(g, tile)) return tile + kTileNarrow;
    // Sixteen wavefronts of 64 x 64 instead of eight of 128 x 64, the same bits, where every unit has several tiles and the epilogue's low-rank
    // operands fit one staging round: 16384 x 5120 outputs at K = 5120 and rank 16, us, eight / sixteen wavefronts: forward 427 / 414, gradient 418 /
    // 397, at 13824 1003 / 980.  One tile for a unit is level or slower (4096 x 4096 at 4096 78.5 / 80.1), rank 64 too (8192 x 11008 455 / 454).
    if (tile == kTile256x256 && g.r <= 16 && !g.accumulate && g.K >= 4096 && ((g.M + 255) / 256) * ((g.N + 255) / 256) > 512)
        return kTile256x256Many;
    // (the same bits; its wavefronts leave half of a compute unit's registers to the weight gradients on the second stream: training step
    // of 2048 x 3072 -> 9216 191.6 us, 214.1 with eight wavefronts of 165 registers)
    return g.beside && tile == kTile128x192Deep ? kTile128x192Beside : tile;
}

hipError_t launch_gemm_one(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    const int tile = product_tile(g, dump_acc);
    if (tile >= kRows16x16) return launch_gemm_rows(g, tile, stream);
    GemmArgs a = g;
    if (tile == kTileSplitSmall2 || tile == kTileSplitSmall4) a.split_scratch = g.small_split_scratch;
    return g.b_layout == kPackedKN ? launch_gemm_kn(a, tile, dump_acc, stream) : launch_gemm_nk(a, tile, dump_acc, stream);
}

const char* gemm_form_name(const GemmArgs& g) {
    static const char* const kNames[] = {"256x256", "256x288", "256x128", "128x192", "128x192 deep", "128x192 beside", "128x128", "64x128", "64x64",
                                         "256x256 many", "256x192 split", "128x192 shared by 2", "128x192 shared by 4", "256x256 narrow",
                                         "256x288 narrow", "256x128 narrow", "", "", "", "", "16x16 rows", "32x32 rows", "32x64 rows", "16x64 rows"};
    static_assert(sizeof(kNames) / sizeof(kNames[0]) == kRows16x64 + 1 && kTileNarrow == 13 && kRows16x16 == 20, "a name for each");
    static thread_local char text[64];
    if (g.K2 <= 128) return kNames[product_tile(g, false)];
    const int wide = choose_wide(g.M, g.N, g.K, g.K2, g.r);
    if (wide >= 0) snprintf(text, sizeof(text), "%s wide", kNames[wide]);
    else snprintf(text, sizeof(text), "%s onto %s", kNames[product_tile(main_product(g), false)], kNames[product_tile(second_product(g), false)]);
    return text;
}

}  // namespace quaff
