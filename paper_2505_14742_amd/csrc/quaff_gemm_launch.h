// Host side of one tile shape of the INT8 MFMA GEMM (quaff_gemm_dma.h): kernel selection and launch.  The two readings of
// the B operand are compiled in translation units of their own (quaff_gemm_fwd.hip, quaff_gemm_bwd.hip).
#pragma once
#include "quaff_gemm_dma.h"

namespace quaff {

// What a tile shape is compiled for beside the fp32 output
constexpr int kFormDump = 1, kFormBf16 = 2, kFormAccumulate = 4, kAllForms = 7;

template <int BM, int BN, int WGM, int WGN, int NS, int MINB, bool BT, bool RAGGED, int KSPLIT, int BK = 128, bool WIDE = false, int FORMS = kAllForms>
static hipError_t launch_dma_form(const GemmArgs& g, bool dump, hipStream_t stream) {
    using C = DmaCfg<BM, BN, WGM, WGN, NS, BK>;
    int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (int)((g.N + BN - 1) / BN);
    TileMap tm = make_tile_map(tiles_m, tiles_n, BM, BN, MINB);
    while ((tm.rm + tm.gm - 1) / tm.gm > 65535) tm.gm *= 2;
    // x % 8 = XCD, x / 8 = tile row inside a group of gm, y = tile column, z = group; a split contraction multiplies y
    // (the parts of a tile are neighbours)
    const int groups = (tm.rm + tm.gm - 1) / tm.gm;
    dim3 grid(8 * (unsigned)tm.gm, (unsigned)tm.rn * KSPLIT, (unsigned)groups), block(C::NT);
    if (tm.rn * KSPLIT > 65535) return hipErrorInvalidValue;
    // the epilogue operands are staged through the idle LDS ring (launch_gemm splits wider second products off)
    if (!dump && !WIDE && (int64_t)(g.K2 / 64) * C::K2_PLANES_BYTES > C::EPI_LIMIT) return hipErrorInvalidValue;
    const size_t lds = dump ? C::LDS_BYTES : C::LDS_ALLOC;
    auto k = gemm_i8_dma_kernel<BM, BN, WGM, WGN, NS, MINB, false, false, false, BT, RAGGED, KSPLIT, BK, WIDE>;
    if constexpr (WIDE) {
        if (dump || g.accumulate || g.C16) return hipErrorInvalidValue;
    } else if constexpr (KSPLIT > 1) {
        if (dump || g.accumulate) return hipErrorInvalidValue;
        if (g.C16) k = gemm_i8_dma_kernel<BM, BN, WGM, WGN, NS, MINB, false, false, true, BT, RAGGED, KSPLIT, BK>;
    } else {
        if (dump) {
            if constexpr (!(FORMS & kFormDump)) return hipErrorInvalidValue;
            else k = gemm_i8_dma_kernel<BM, BN, WGM, WGN, NS, MINB, true, false, false, BT, RAGGED, 1, BK>;
        } else if (g.C16) {
            if constexpr (!(FORMS & kFormBf16)) return hipErrorInvalidValue;
            else k = gemm_i8_dma_kernel<BM, BN, WGM, WGN, NS, MINB, false, false, true, BT, RAGGED, 1, BK>;
        } else if (g.accumulate) {
            // (only a forward product has a wide second product to accumulate onto)
            if constexpr (BT || !(FORMS & kFormAccumulate)) return hipErrorInvalidValue;
            else k = gemm_i8_dma_kernel<BM, BN, WGM, WGN, NS, MINB, false, true, false, BT, RAGGED, 1, BK>;
        }
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, grid, block, lds, stream, g, tm);
    return hipGetLastError();
}

// BM x BN tile, WGM x WGN wavefronts, NS stages in the ring, MINB workgroups per compute unit to compile for
template <int BM, int BN, int WGM, int WGN, int NS, int MINB, bool BT, int FORMS = kAllForms>
static hipError_t launch_dma(const GemmArgs& g, bool dump, hipStream_t stream) {
    if (g.K % 128 != 0) return launch_dma_form<BM, BN, WGM, WGN, NS, MINB, BT, true, 1, 128, false, FORMS>(g, dump, stream);
    return launch_dma_form<BM, BN, WGM, WGN, NS, MINB, BT, false, 1, 128, false, FORMS>(g, dump, stream);
}

}  // namespace quaff
