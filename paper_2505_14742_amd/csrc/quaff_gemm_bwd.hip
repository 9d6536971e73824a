// INT8 MFMA GEMM with the B operand read as [K x N] from the packed weight codes (the input-gradient product).
#include "quaff_gemm_launch.h"

namespace quaff {

hipError_t launch_gemm_kn(const GemmArgs& g, int tile, bool dump_acc, hipStream_t stream) {
    switch (tile) {
        case kTile256x256: return launch_dma<256, 256, 2, 4, 2, 1, true>(g, dump_acc, stream);
        case kTile256x256Many: return launch_dma<256, 256, 4, 4, 2, 1, true>(g, dump_acc, stream);
        case kTile256x288: return launch_dma<256, 288, 4, 3, 2, 1, true>(g, dump_acc, stream);
        case kTile256x128: return launch_dma<256, 128, 4, 2, 2, 1, true>(g, dump_acc, stream);
        case kTile128x192: return launch_dma<128, 192, 2, 2, 2, 2, true>(g, dump_acc, stream);
        case kTile128x192Deep: return launch_dma<128, 192, 4, 2, 3, 2, true>(g, dump_acc, stream);
        case kTile128x192Beside: return launch_dma<128, 192, 2, 2, 3, 2, true, 0>(g, dump_acc, stream);      // (of the backward step only)
        case kTile128x128: case kTile64x128: case kTile64x64: return launch_gemm_mid(g, tile, dump_acc, stream);
        case kTileSplit: return launch_dma_form<256, 192, 4, 2, 2, 1, true, false, 2>(g, dump_acc, stream);
        case kTileSplitSmall2: return launch_dma_form<128, 192, 2, 2, 3, 2, true, false, 2>(g, dump_acc, stream);
        case kTileSplitSmall4: return launch_dma_form<128, 192, 2, 2, 3, 2, true, false, 4>(g, dump_acc, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace quaff
