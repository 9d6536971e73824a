// INT8 MFMA GEMM of the forward product with a second product of more than 128 columns (the paper's outlier budgets) in the same
// launch: a main loop over xq_O and what_int of its own, then the one over the codes, two sets of accumulators.  Tiles with at most
// three 32 x 32 blocks to a wavefront have the registers for it.  As two launches the output is written, read and written again:
// 2048 x 8192 -> 3072 with 819 outliers 14.3 + 60.6 us, 62 in one (128 x 192 tiles).
#include "quaff_gemm_launch.h"

namespace quaff {

template <int BM, int BN, int WGM, int WGN>
static hipError_t launch_wide(const GemmArgs& g, hipStream_t stream) {
    if (g.K % 128 != 0) return launch_dma_form<BM, BN, WGM, WGN, 3, 2, false, true, 1, 128, true>(g, false, stream);
    return launch_dma_form<BM, BN, WGM, WGN, 3, 2, false, false, 1, 128, true>(g, false, stream);
}

hipError_t launch_gemm_wide(const GemmArgs& g, int tile, hipStream_t stream) {
    switch (tile) {
        case kTile128x192Deep: return launch_wide<128, 192, 4, 2>(g, stream);
        case kTile128x128: return launch_wide<128, 128, 4, 2>(g, stream);
        case kTile64x128: return launch_wide<64, 128, 2, 4>(g, stream);
        case kTile64x64: return launch_wide<64, 64, 2, 2>(g, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace quaff
