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

namespace quaff {

namespace {
// Shapes a product can take, and the time of each, estimated in us:
//   fixed + round ((n - 1) / fit) + next (n - 1) + n ((bm + bn) K (kb + busy b) 1e-6 + lora rank')
// with n the tiles of the busiest compute unit (an XCD's region of the tile grid over its 32 units, rounded up), fit the
// workgroups of the shape that are resident on a unit together, b the share of the units that have a tile, and rank' the 32-column
// rounds of the adapter's staged operands or, for the shapes of quaff_gemm_rows.hip, which fetch them block by block,
// (rank / 16)^2.  (bm + bn) K are the operand bytes of a tile: what bounds every shape is their delivery, 55 to 85 KB/us to one
// compute unit and less of it with all units busy.
// The constants are fitted to 1178 products (20 to 6000 rows, 64 to 16384 columns, contractions of 208 to 14000, ranks 0 to 64,
// 0 to 100 outliers; launch alone, every shape timed).  The shape chosen takes 1.013 (forward) and 1.010 (input gradient) of the time of
// the best one in the geometric mean, at worst 1.42 (320 x 9088 at K = 256: 64 x 64 tiles for 128 x 128).  Without the three shapes
// of 64 and 128 rows the same choice takes 1.22 and 1.29: one of the wider ones leaves most units idle or walks
// the contraction alone on a few (us, before / now: 1003 x 2064 at 1040 15.1 / 10.0, 2048 x 1024 at 3072 19.3 / 12.2,
// 768 x 1536 at 1536 13.7 / 7.8, gradient 1003 x 1040 at 2064 with its quantizer 26.0 / 15.3).
struct Shape { int id, bm, bn, fit; double fixed, round, next, kb, busy, lora; };
constexpr Shape kForward[10] = {
    {kTile256x256, 256, 256, 1, 10.67, 8.75, 3.70, 15.58, 6.01, 2.96},
    {kTile256x288, 256, 288, 1, 10.01, 11.07, 4.79, 17.48, 5.89, 3.00},
    {kTile256x128, 256, 128, 1, 7.69, 6.87, 3.05, 13.31, 5.20, 1.90},
    {kTile128x192, 128, 192, 2, 8.69, 8.82, 0.00, 8.89, 6.71, 1.77},       // more tiles than units
    {kTile128x128, 128, 128, 1, 5.50, 3.60, 1.12, 12.43, 3.68, 0.96},
    {kTile64x128, 64, 128, 2, 4.36, 2.11, 0.91, 11.60, 1.45, 0.51},
    {kTile64x64, 64, 64, 3, 4.40, 2.17, 0.12, 14.44, 0.00, 0.39},
    {kRows32x64, 32, 64, 4, 4.29, 0.99, 1.67, 15.61, 1.90, 0.20},
    {kRows32x32, 32, 32, 8, 3.56, 3.95, 0.36, 17.59, 1.69, 0.10},
    {kRows16x16, 16, 16, 8, 3.21, 0.75, 0.53, 17.28, 0.00, 0.04}};
constexpr Shape kGradient[9] = {
    {kTile256x256, 256, 256, 1, 9.11, 10.04, 0.00, 15.96, 5.69, 3.00},
    {kTile256x288, 256, 288, 1, 9.07, 10.46, 4.51, 16.95, 5.99, 3.00},
    {kTile256x128, 256, 128, 1, 5.92, 4.85, 1.86, 13.42, 4.89, 2.24},
    {kTile128x192, 128, 192, 2, 5.64, 2.32, 2.27, 8.62, 6.34, 1.94},       // more tiles than units
    {kTile128x128, 128, 128, 1, 4.73, 3.13, 1.07, 12.78, 3.56, 1.18},
    {kTile64x128, 64, 128, 2, 3.93, 2.08, 0.57, 12.19, 0.79, 0.68},
    {kTile64x64, 64, 64, 3, 4.28, 2.23, 0.00, 13.43, 0.00, 0.46},
    {kRows32x64, 32, 64, 4, 4.73, 10.03, 0.74, 13.88, 3.24, 0.19},
    {kRows16x64, 16, 64, 2, 4.10, 0.00, 2.82, 9.55, 3.47, 0.11}};
// The 128 x 192 tile with at most one tile for every unit takes a ring of three stages (120 KB of LDS: one workgroup per unit) and
// eight wavefronts.  The third stage keeps the operands of the stage after next in flight, which is what a product whose operands
// come from HBM rather than from the Infinity Cache needs (back to back on operand sets that rotate through more than the
// cache holds, two stages / three: o_proj forward 36.2 / 30.5 us, qkv dX 79.2 / 69.8, 8192 -> 3072 forward 74.1 / 61.7; on cached
// operands level).  Eight wavefronts of 32 x 96 against four of 64 x 96: 2048 x 3072 outputs 26.3 / 27.5 us at K = 3072, 55.9 / 57.8 at
// 8192, level at 9216; gradient with its quantizer 34.7 / 36.5, 71.7 / 71.6; 2048 x 2176 at 768 and similar 0.8 of the time.  With more
// tiles than units two workgroups per unit overlap each other's epilogues instead, which needs the smaller ring and four wavefronts
// (4480 x 13376 at 576, rank 64: 115 us, 134 with the deep ring).
constexpr Shape kDeep[2] = {{kTile128x192Deep, 128, 192, 1, 6.69, 4.59, 1.80, 12.68, 4.17, 1.26},
                            {kTile128x192Deep, 128, 192, 1, 5.83, 4.04, 1.49, 13.27, 3.81, 1.42}};

double shape_us(const Shape& s, int64_t M, int64_t N, int64_t K, int32_t rank) {
    // (32-bit divisions: M is below 2^30, N below 2^20)
    const uint32_t tm = ((uint32_t)M + s.bm - 1) / (uint32_t)s.bm, tn = ((uint32_t)N + s.bn - 1) / (uint32_t)s.bn;
    const int64_t tiles = (int64_t)tm * tn;
    int64_t n = (tiles + 255) / 256;
    if (n <= 16) {                    // (with many tiles per unit the regions' edges don't matter)
        const TileGrid r = tile_grid((int)tm, (int)tn, s.bm, s.bn);
        n = ((int64_t)r.rm * r.rn + 31) / 32;
    }
    const double busy = tiles < 256 ? (double)tiles / 256.0 : 1.0;
    const int columns = s.id >= kRows16x16 ? (rank / 16) * (rank / 16) : (rank + 31) / 32;
    return s.fixed + s.round * (double)((n - 1) / s.fit) + s.next * (double)(n - 1) +
           (double)n * ((s.bm + s.bn) * (double)K * 1e-6 * (s.kb + s.busy * busy) + s.lora * columns);
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
// exchange of their sums through the L2.  Estimated in the terms of choose_shape (`k` = 1024 of contraction, `busy` = tiles per
// compute unit); 4 % must be gained over the best unshared shape, which happens from K = 8192 on.  One workgroup per tile in its
// best shape / two or four, us: forward 1098 x 2048 outputs at 8192 35.4 / 34.3, 763 x 1408 at 14336 37.8 / 33.8 (four), 479 x 2176 at
// 16384 44.4 / 35.4, 2021 x 1152 at 16384 61.5 / 52.6; input gradient with its quantizer 970 x 2944 <- 16384 83.8 / 78.4.
// The workgroups of a tile run on one XCD and one of them fills a compute unit: no more of them than the 32 units of an XCD,
// or the last tiles start when the first have ended (1408 x 2112 outputs, 11 x 11 tiles, 18 of them on an XCD, one / two
// workgroups per tile: 27.8 / 40.1 us at K = 4096, 45.1 / 58.1 at 8192; 640 x 2048 outputs, one / four: 25.6 / 30.5 at 4096).
static int small_split(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient, double gain = 1.04) {
    const int64_t tiles = ((M + 127) / 128) * ((N + 191) / 192);
    if (tiles > 128 || K % 256 != 0 || K < 6144) return 1;      // (nothing is gained below: no need to estimate)
    double alone;
    choose_shape(M, N, K, rank, gradient, &alone);
    const double k = (double)K / 1024.0, busy = tiles / 256.0;
    const double two = gain * (9.7 + 6.5 * busy + (2.2 + 1.6 * busy) * k);
    const double four = gain * (11.0 + 13.0 * busy + (1.15 + 3.1 * busy) * k);
    // (tiles on the busiest XCD: the grid is cut into eight regions of equal size, rounded up)
    const TileMap map = make_tile_map((int)((M + 127) / 128), (int)((N + 191) / 192), 128, 192, 1);
    const int on_xcd = map.rm * map.rn;
    if (4 * on_xcd <= 32 && K % 512 == 0 && four < alone && four < two) return 4;
    return 2 * on_xcd <= 32 && two < alone ? 2 : 1;
}
// Beside the weight gradients of rank 32 and more on a second stream, whose workgroups (88 to 106 KB of LDS) leave no room on a
// compute unit for one of these, some wait for a partner that has no unit yet: 15 % must be gained.  Backward steps with a second
// stream, us, shared / not: 2998 x 896 <- 3840 at rank 32 74.7 / 67.8, at rank 64 80.3 / 72.1, 2048 x 1536 <- 4096 at rank 32 68.3 /
// 64.0 (expected gain 4 %); 512 x 3072 <- 3072 at rank 32 46.0 / 50.3 (15 %), 1024 x 2048 <- 8192 78.6 / 92.4 (30 %).
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

hipError_t launch_gemm(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    ProfScope prof(K_GEMM, stream);
    // (two launches: the first writes row_scale * acc2 * col_scale2, the main product accumulates onto it)
    // bf16 output exists in the single-launch form only
    if (g.C16 && (g.K2 > 128 || dump_acc)) return hipErrorNotSupported;
    if (!dump_acc && g.K2 > 128) {
        const int wide = choose_wide(g.M, g.N, g.K, g.K2, g.r);
        if (wide >= 0) return launch_gemm_wide(g, wide, stream);
        GemmArgs c2{};
        c2.A = g.A2; c2.lda = g.K2; c2.B = g.B2; c2.ldb = g.K2;
        c2.M = g.M; c2.N = g.N; c2.K = g.K2;
        c2.row_scale = g.row_scale; c2.col_scale = g.col_scale2;
        c2.C = g.C; c2.ldc = g.ldc;
        hipError_t e = launch_gemm_one(c2, false, stream);
        if (e != hipSuccess) return e;
        GemmArgs m = g;
        m.K2 = 0; m.A2 = nullptr; m.B2 = nullptr; m.col_scale2 = nullptr;
        m.accumulate = 1;
        return launch_gemm_one(m, false, stream);
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

// Which kernel a product with an adapter takes depends on its sizes alone, not on the type of its output and not on the room
// in the workspace: the kernels add the low-rank term in different orders, and a call's last bits may not depend on either.
hipError_t launch_gemm_one(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    const bool gradient = g.b_layout == kPackedKN, one_launch = !dump_acc && !g.accumulate && g.K2 <= 128;
    const int parts = one_launch ? small_split(g.M, g.N, g.K, g.r, gradient) : 1;
    int tile;
    if (g.split_scratch && one_launch && split_applies(g.M, g.N, g.K)) {
        tile = kTileSplit;
    } else if (parts > 1 && g.small_split_scratch) {
        GemmArgs split = g;
        split.split_scratch = g.small_split_scratch;
        tile = parts == 2 ? kTileSplitSmall2 : kTileSplitSmall4;
        return gradient ? launch_gemm_kn(split, tile, false, stream) : launch_gemm_nk(split, tile, false, stream);
    } else if (parts > 1 && g.r > 0) {
        tile = kTile128x192;             // (no room for the exchange: the shared form's tile and epilogue, one workgroup each)
    } else {
        double us;
        tile = choose_shape(g.M, g.N, g.K, g.r, gradient, &us);
        if (tile >= kRows16x16) return launch_gemm_rows(g, tile, stream);
    }
    if (!gradient && narrow_stages(g, tile)) tile += kTileNarrow;
    // Sixteen wavefronts of 64 x 64 instead of eight of 128 x 64, the same bits, where every unit has several tiles and the epilogue's low-rank
    // operands fit one staging round: 16384 x 5120 outputs at K = 5120 and rank 16, us, eight / sixteen wavefronts: forward 427 / 414, gradient 418 /
    // 397, at 13824 1003 / 980.  One tile for a unit is level or slower (4096 x 4096 at 4096 78.5 / 80.1), rank 64 too (8192 x 11008 455 / 454).
    if (tile == kTile256x256 && g.r <= 16 && !g.accumulate && g.K >= 4096 && ((g.M + 255) / 256) * ((g.N + 255) / 256) > 512)
        tile = kTile256x256Many;
    // (the same bits; its wavefronts leave half of a compute unit's registers to the weight gradients on the second stream: training step
    // of 2048 x 3072 -> 9216 191.6 us, 214.1 with eight wavefronts of 165 registers)
    if (g.beside && tile == kTile128x192Deep) tile = kTile128x192Beside;
    return gradient ? launch_gemm_kn(g, tile, dump_acc, stream) : launch_gemm_nk(g, tile, dump_acc, stream);
}

}  // namespace quaff
