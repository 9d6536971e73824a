// INT8 MFMA GEMM, the tiles of 64 and 128 rows for outputs that give the wide ones too few tiles (quaff_gemm.hip chooses), in
// both readings of B.  Many wavefronts for their size (32 x 32 of the output each, 32 x 64 in the largest tile): they share the
// issue of the direct loads and the epilogue, which are what such a launch consists of beside the delivery of its operands.
// Us, 64 x 128 tile with four / eight wavefronts: 512 x 3072 outputs at K = 3072 14.9 / 11.7, 2048 x 1024 at 3072 14.6 / 12.2; 128 x 128
// tile: 1003 x 2064 at 1040 11.8 / 10.0, 1536 x 2048 at 2048 13.8 / 13.0.  (Their accumulating forms are reached by contractions beyond 16384
// columns only: 134 x 32944 -> 10976 with 170 outliers.)
#include "quaff_gemm_launch.h"

namespace quaff {

template <bool BT>
static hipError_t launch_mid(const GemmArgs& g, int tile, bool dump_acc, hipStream_t stream) {
    switch (tile) {
        case kTile128x128: return launch_dma<128, 128, 4, 2, 3, 2, BT>(g, dump_acc, stream);
        case kTile64x128: return launch_dma<64, 128, 2, 4, 3, 2, BT>(g, dump_acc, stream);
        case kTile64x64: return launch_dma<64, 64, 2, 2, 3, 2, BT>(g, dump_acc, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_mid(const GemmArgs& g, int tile, bool dump_acc, hipStream_t stream) {
    return g.b_layout == kPackedKN ? launch_mid<true>(g, tile, dump_acc, stream) : launch_mid<false>(g, tile, dump_acc, stream);
}

}  // namespace quaff
