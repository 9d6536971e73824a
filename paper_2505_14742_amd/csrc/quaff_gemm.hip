// INT8 MFMA GEMM with int32 accumulation and a fused dequantising epilogue (Eq. 9 of the paper) that also
// adds the rank-r LoRA term.  The same kernels serve the forward product (contraction over c_in) and the
// input-gradient product (contraction over c_out).  A is contraction-contiguous; B is either a plain
// contraction-contiguous [N x K] matrix or the packed weight codes (one copy, quaff_internal.h), read as [N x K] by
// the forward product and as [K x N], through transposing LDS reads, by the input-gradient product.
//
//   C[i, j] = row_scale[i] * ( acc1[i, j] * col_scale[j] + acc2[i, j] * col_scale2[j] ) + sum_p T[i, p] L[j, p]
//   acc1 = A B^T   (K long, the hot loop),   acc2 = A2 B2^T   (K2 = padded outlier count, done in the epilogue)
//
// One kernel template (quaff_gemm_dma.h) serves every shape: direct-to-LDS operand streaming through a ring of stages,
// v_mfma_i32_32x32x32_i8, XCD-aware tile order; this file chooses the tile shape.
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
int choose_tile(int64_t M, int64_t N) {
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

hipError_t launch_gemm_one(const GemmArgs& g, bool dump_acc, hipStream_t stream) {
    int tile;
    if (g.split_scratch && !dump_acc && !g.C16 && !g.accumulate && g.K2 <= 128 && split_applies(g.M, g.N, g.K))
        tile = kTileSplit;
    else
        tile = choose_tile(g.M, g.N);
    // The 128 x 192 tile with at most one tile per compute unit takes a ring of three stages (120 KB of LDS: one
    // workgroup per unit): the operands of the stage after next are then in flight too, which is what a product whose
    // operands come from HBM rather than from the Infinity Cache needs (measured back to back on operand sets that
    // rotate through more than the cache holds: o_proj forward 36.2 -> 30.5 us, qkv dX 79.2 -> 69.8, 8192 -> 3072
    // forward 74.1 -> 61.7; on cached operands the two rings are level, 29.4 / 65.6 / 60.1 us).  It is compiled for
    // the register budget of two workgroups per unit like the two-stage form (with the whole file to itself the
    // compiler's schedule is 2 - 8 % slower).  With more tiles than units two workgroups per unit overlap each
    // other's epilogues instead, which needs the smaller ring.
    if (tile == kTile128x192 && ((g.M + 127) / 128) * ((g.N + 191) / 192) <= 256) tile = kTile128x192Deep;
    return g.b_layout == kPackedKN ? launch_gemm_kn(g, tile, dump_acc, stream) : launch_gemm_nk(g, tile, dump_acc, stream);
}

}  // namespace quaff
