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
// Tile shapes.  `spc` = workgroups that fit on one compute unit at once (LDS and registers);
// `ineff` = measured cost per MAC relative to the 256x256 shape on a large problem.
struct TileChoice { int bm, bn, spc; double ineff; };
constexpr TileChoice kChoices[4] = {
    {256, 256, 1, 1.00},   // 8 wavefronts, 128x64 each
    {256, 288, 1, 1.03},   // 12 wavefronts, 64x96 each: 2048 x 9216 outputs are exactly 256 such tiles
    {256, 128, 1, 1.18},   // 8 wavefronts, 64x64 each (its wide-stage ring leaves room for one workgroup per unit)
    {128, 192, 2, 1.20},   // 4 wavefronts, 64x96 each: 2048 x 3072 outputs are exactly 256 such tiles
};

// Estimated time of a tile shape on 256 compute units: full rounds of spc tiles per unit, then the remainder at one
// tile per unit per pass.  The shape that wastes the fewest compute-unit passes wins.
int choose_tile(int64_t M, int64_t N, double* best_work) {
    int best = 0;
    double best_cost = -1.0;
    for (int c = 0; c < 4; ++c) {
        const TileChoice& t = kChoices[c];
        int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        int64_t slots = 256 * t.spc;
        int64_t full = tiles / slots, rem = tiles % slots;
        double passes = (double)full * t.spc + (double)((rem + 255) / 256);
        double cost = passes * t.bm * t.bn * t.ineff;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = c; }
    }
    *best_work = best_cost;
    return best;
}

// Small outputs.  Estimated time of a shape of quaff_gemm_rows.hip: launch and epilogue, then the slower of the two ways its
// operands arrive - one compute unit's share at `cu_rate`, or all of it at `chip_rate` - and 1.5 us for every further
// round of 256 tiles (their epilogues do not overlap their loads).  Against it stand, per 1024 bytes of contraction, 4.4 us (6.1
// with every compute unit busy) per pass of 128 x 192 tiles and 8 us; 7 where tiles without an edge have little to multiply
// (768 x 1536 and 384 x 3072 outputs, large tiles / 32 x 64 tiles: forward 8.2 / 9.5 us at K = 256, 10.5 / 11.3 at 768; input
// gradient with its quantizer 9.6 / 11.6 at 256, 10.9 / 12.3 at 512; with edges, 722 x 1776 outputs at 256, 10.0 / 9.6).  The
// factor 1.1 keeps close calls with the large tiles.  Over 2388 products of 1 to 2500 rows, 64 to 12000 columns and 128 to 14000
// contractions, every shape and split timed, the choice takes 0.45 (forward) and 0.62 (input gradient, quantizer included) of
// the time of the large tiles in the geometric mean; one is more than 2 % slower than them (575 x 2080 at 512: 12.4 / 12.0).
// Against the best of all shapes it is 1.4 % slower in the mean and more than 20 % in 46, most of them long
// contractions for which the 64 x 96 tile is taken for faster than it is (256 x 2048 at 8192: 31.5 us, 32 x 64 tiles 18.9).
// An adapter of a high rank is fetched and multiplied block by block here, in one pass over staged operands there: with a short
// contraction and more than `lora_from` rounds the small tiles lose lora_us for every further round and (rank / 16)^2 - 1.  From
// 600 products timed at rank 0 and at 16, 32 or 64 in every shape, and 500 in the shape chosen here and with the large tiles: at
// rank 64 and 2 to 3 rounds of 32 x 64 tiles the loss is 7.5 us forward and 4.6 in the gradient (700 x 1936 gradient at K = 128,
// large tiles / 32 x 64 tiles: 16.8 / 24.7 us; 132 x 8480 at 192 and rank 32 12.5 / 17.4), at rank 16 level, and beyond K = 768 the
// small tiles are ahead all the same (3889 x 256 gradient at 1664 and rank 48: 33.3 / 30.1).  Of 1700 products with an adapter or
// more than one round 22 are still more than 2.5 % slower than the large tiles; without this term 60 are.
struct RowsChoice { int shape, bm, bn; double fixed_us, cu_rate, chip_rate, lora_us, lora_from; };   // rates in KB/us and MB/us
constexpr RowsChoice kRowsForward[4] = {
    {kRows16x16, 16, 16, 3.2, 83, 11.5, 0.0, 1.0}, {kRows32x32, 32, 32, 3.6, 79, 10.2, 0.0, 1.0},
    {kRows32x64, 32, 64, 4.4, 84, 10.1, 0.5, 1.5}, {kRows64x96, 64, 96, 7.9, 80, 7.7, 0.9, 0.4}};
constexpr RowsChoice kRowsGradient[2] = {{kRows16x64, 16, 64, 4.0, 115, 11, 0.12, 1.5}, {kRows32x64, 32, 64, 4.5, 85, 10.1, 0.5, 1.5}};

int choose_rows(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient, double tile_work, double* us_estimate) {
    const double passes = tile_work / (128.0 * 192.0 * kChoices[kTile128x192].ineff);
    const int64_t wide_tiles = ((M + 127) / 128) * ((N + 191) / 192);
    const double busy = wide_tiles < 256 ? wide_tiles / 256.0 : 1.0;
    const bool short_and_whole = K <= 1024 && M % 128 == 0 && N % 192 == 0;
    double best_us = ((short_and_whole ? 7.0 : 8.0) + (double)K * 1e-3 * passes * (4.4 + 1.75 * busy)) / 1.1;
    int best = kRowsNone;
    for (int c = 0; c < (gradient ? 2 : 4); ++c) {
        const RowsChoice& r = gradient ? kRowsGradient[c] : kRowsForward[c];
        const double tiles = (double)((M + r.bm - 1) / r.bm) * (double)((N + r.bn - 1) / r.bn);
        const double tile_kb = (r.bm + r.bn) * (double)K * 1e-3, rounds = tiles / 256.0;
        const double per_cu = tile_kb * (rounds > 1.0 ? __builtin_ceil(rounds) : 1.0) / r.cu_rate, chip = tile_kb * tiles * 1e-3 / r.chip_rate;
        const double lora = rank > 16 && K <= 768 && rounds > r.lora_from ? r.lora_us * (rounds - r.lora_from) * ((rank / 16) * (rank / 16) - 1) : 0.0;
        const double us = r.fixed_us + (per_cu > chip ? per_cu : chip) + (rounds > 1.0 ? 1.5 * (rounds - 1.0) : 0.0) + lora;
        if (us < best_us) { best_us = us; best = r.shape; }
    }
    *us_estimate = best_us;
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

// Outputs of at most 128 tiles of 128 x 192 leave half of the compute units idle or more while every tile walks its
// contraction alone; two or four workgroups per tile share it where that pays for the exchange of their sums through the L2.
// Estimated in the terms of choose_rows (`k` = 1024 of contraction, `busy` = tiles per compute unit); 4 % must be gained.
// Of 1815 products with at most 128 tiles and whole stages, timed every way, 191 are shared: 0.86 of the time of the best unshared
// shape in the geometric mean, 24 of them slower than it by more than 3 % (18 % at most); 23 others would gain more than 5 %.
// Forward, one / two / four workgroups per tile, us: 512 x 3072 outputs 19.7 / 17.0 / 18.3 at K = 3072, 43.3 / 29.0 / 26.2 at 8192,
// 10.6 / 11.6 / 13.1 at 1024; 1024 x 3072 outputs 20.2 / 20.7 at 3072, 44.0 / 34.7 at 8192; 256 x 3072 outputs at 8192 30.6 (64 x 96
// tiles) / 27.6 / 21.6.  Input gradient with its quantizer: 512 x 3072 <- 3072 27.3 / 23.9 / 25.4, <- 8192 52.9 / 36.6 / 32.6.
// The workgroups of a tile run on one XCD and one of them fills a compute unit: no more of them than the 32 units of an XCD,
// or the last tiles start when the first have ended (1408 x 2112 outputs, 11 x 11 tiles, 18 of them on an XCD, one / two
// workgroups per tile: 27.8 / 40.1 us at K = 4096, 45.1 / 58.1 at 8192; 640 x 2048 outputs, one / four: 25.6 / 30.5 at 4096).
static int small_split(int64_t M, int64_t N, int64_t K, int32_t rank, bool gradient, double gain = 1.04) {
    const int64_t tiles = ((M + 127) / 128) * ((N + 191) / 192);
    if (tiles > 128 || K % 256 != 0) return 1;
    double work, best_us;
    choose_tile(M, N, &work);
    const double k = (double)K / 1024.0, busy = tiles / 256.0;
    double alone = 8.1 + 4.7 * k;
    if (choose_rows(M, N, K, rank, gradient, work, &best_us) != kRowsNone && best_us < alone) alone = best_us;
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

hipError_t launch_gemm(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    ProfScope prof(K_GEMM, stream);
    // A second product too wide for the epilogue's LDS staging (more than two 64-wide outlier slices) runs as a launch
    // of its own that writes row_scale * acc2 * col_scale2, and the main product then accumulates onto it: one extra
    // write and read of the output instead of a slow epilogue.
    // bf16 output exists in the single-launch form only
    if (g.C16 && (g.K2 > 128 || dump_acc)) return hipErrorNotSupported;
    if (!dump_acc && g.K2 > 128) {
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
// zeros.  Forward products, us, 64 / 128 bytes: 2048 x 3072 outputs (128 x 192 tiles) 8.2 / 9.2 at K = 192, 10.8 / 11.5 at 576, 12.5 /
// 12.8 at 832 (2048 x 1024 there 11.4 / 11.1), 14.0 / 14.0 at 1088, 20.7 / 19.9 at 2112; 4096 x 8192 outputs (256 x 256) 27.9 / 29.3 at
// 192, 44.9 / 46.0 at 832, 52.0 / 51.5 at 1088, 140.9 / 136.7 at 4160.  The 256 x 128 tile has room for two workgroups on a compute
// unit with the narrow ring and gains at any length: 8192 x 3072 21.9 / 25.4 at 192, 64.8 / 70.3 at 2112, 112.8 / 119.0 at 4160.
// Not with outliers on the two largest tiles: their epilogue's operands fit side by side in the wide ring only (2423 x 320 -> 5536,
// rank 16: 23.0 / 17.6; forward step of 4712 x 960 -> 15360 at rank 0: 170 / 154).
static bool narrow_stages(const GemmArgs& g, int tile) {
    if (g.K % 128 != 64 || tile > kTile128x192) return false;
    if (tile == kTile256x128) return true;
    return tile == kTile128x192 ? g.K < 768 : g.K < 1024 && g.K2 == 0;
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
        double work, us;
        tile = choose_tile(g.M, g.N, &work);
        const int rows = choose_rows(g.M, g.N, g.K, g.r, gradient, work, &us);
        if (rows != kRowsNone) return launch_gemm_rows(g, rows, stream);
    }
    // The 128 x 192 tile with at most one tile per compute unit takes a ring of three stages (120 KB of LDS: one
    // workgroup per unit): the operands of the stage after next are then in flight too, which is what a product whose
    // operands come from HBM rather than from the Infinity Cache needs (measured back to back on operand sets that
    // rotate through more than the cache holds: o_proj forward 36.2 -> 30.5 us, qkv dX 79.2 -> 69.8, 8192 -> 3072
    // forward 74.1 -> 61.7; on cached operands the two rings are level, 29.4 / 65.6 / 60.1 us).  It is compiled for
    // the register budget of two workgroups per unit like the two-stage form (with the whole file to itself the
    // compiler's schedule is 2 - 8 % slower).  With more tiles than units two workgroups per unit overlap each
    // other's epilogues instead, which needs the smaller ring.
    if (!gradient && narrow_stages(g, tile))
        tile += kTileNarrow;
    else if (tile == kTile128x192 && ((g.M + 127) / 128) * ((g.N + 191) / 192) <= 256) tile = kTile128x192Deep;
    return gradient ? launch_gemm_kn(g, tile, dump_acc, stream) : launch_gemm_nk(g, tile, dump_acc, stream);
}

}  // namespace quaff
