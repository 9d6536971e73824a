// INT8 MFMA GEMM for outputs with too few tiles of the large shapes to fill the chip (quaff_gemm_dma.h): few rows, or a few
// hundred rows by a few hundred columns.  See quaff_gemm.hip for the computation and for the rule that chooses.
//
// What bounds such a product is how fast its operands arrive and the length of the dependent chain from launch to last store,
// not the matrix cores.  So the tile is small (MB x NB blocks of 16 x 16), the NW wavefronts of a workgroup share
// the CONTRACTION instead of the tile - wavefront w takes the 64-byte steps w, w + NW, ... of all the tile's rows and
// columns, so that every operand byte is fetched exactly once per workgroup, straight into MFMA fragments, with D steps in
// flight per wavefront and no barrier before the end - and the int32 partial sums meet in LDS (exact in any order).  Block b
// of a round is then finished by wavefront b, whose epilogue operands were requested before the exchange.
// Measured (one launch, us, the 128 x 192 tile with its ring of stages / this kernel): 16 x 3072 -> 9216 forward 21.4 / 7.8 (28 MB
// of codes at 3.6 TB/s), 16 x 8192 -> 3072 44.5 / 8.0, 64 x 3072 -> 3072 22.8 / 7.4, 256 x 3072 -> 3072 20.9 / 15.9,
// 16 x 512 -> 512 9.4 / 3.4; input gradient 16 x 3072 <- 9216 50.5 / 16.1, 64 x 3072 <- 3072 21.9 / 7.1.
// A step of 128 bytes (whole lines of A, lanes exchanging halves) was no faster.
#include "quaff_gemm_dma.h"

namespace quaff {

template <int MB, int NB, int NW, int D, bool BT>
struct RowsCfg {
    static constexpr int BM = MB * 16, BN = NB * 16, NT = NW * 64, BLOCKS = MB * NB;
    static constexpr int PER_ROUND = BLOCKS < NW ? BLOCKS : NW, ROUNDS = BLOCKS / PER_ROUND;
    static constexpr int EXCHANGE_BYTES = NW * PER_ROUND * 1024;
    static constexpr int TR_BYTES = BT ? NW * 4096 : 0;            // transposition buffer of every wavefront (64 x 64 bytes)
    static constexpr int LDS_BYTES = EXCHANGE_BYTES > TR_BYTES ? EXCHANGE_BYTES : TR_BYTES;
    static_assert(BLOCKS % PER_ROUND == 0 && LDS_BYTES <= 65536, "whole rounds, no LDS attribute needed");
    static_assert(!BT || NB == 4, "the transposed operand is fetched in lines of 64 columns");
};

// The two operands are exchanged in the MFMA (the weight's 16 columns are its rows): a lane then holds four neighbouring
// columns of one output row and stores them at once.
template <int MB, int NB, int NW, int D, bool BT>
__global__ void __launch_bounds__(NW * 64)
gemm_i8_rows_kernel(const GemmArgs g, const TileMap tmap) {
    using C = RowsCfg<MB, NB, NW, D, BT>;
    extern __shared__ __attribute__((aligned(1024))) int8_t lds_raw[];
    lds_i8* const lds = (lds_i8*)lds_raw;
    int tile_m, tile_n;
    if (!tile_of_block(tmap, blockIdx.x, blockIdx.y, blockIdx.z, tile_m, tile_n)) return;
    if constexpr (!BT)
        if (g.clear_bytes > 0) clear_words(g, tile_m * tmap.tiles_n + tile_n, tmap.tiles_m * tmap.tiles_n, C::NT);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int64_t m0 = (int64_t)tile_m * C::BM, n0 = (int64_t)tile_n * C::BN;
    const int last_m = (int)((g.M - 1 - m0) < C::BM - 1 ? (g.M - 1 - m0) : C::BM - 1);
    const int last_n = (int)((g.N - 1 - n0) < C::BN - 1 ? (g.N - 1 - n0) : C::BN - 1);

    // Operand addresses: 32-bit lane offsets from the tile's first row; rows past the edge repeat the last one (never stored).
    // A step is 64 bytes of the contraction.  A: MB fetches of 16 rows x 64 bytes.  B: NB fetches of the same shape (packed
    // codes: 8 whole lines each); BT: 4 fetches of 8 whole lines, each 64 columns of two contraction rows.
    const int8_t* const tileA = g.A + m0 * g.lda;
    uint32_t offA[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int row = i * 16 + l16 < last_m ? i * 16 + l16 : last_m;
        offA[i] = (uint32_t)row * (uint32_t)g.lda + quad * 16;
    }
    const bool packed = g.b_layout != kPlain;
    const int8_t* const tileB = BT ? g.B + n0 * 2 : g.B + n0 * g.ldb;      // (BT: n0 is a multiple of 64)
    const int64_t stepB = BT ? 64 * g.ldb : packed ? 128 : 64;
    uint32_t offB[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if constexpr (BT) {
            offB[j] = (uint32_t)(j * 8 + (lane >> 3)) * (uint32_t)(2 * g.ldb) + (lane & 7) * 16;
        } else {
            const int row = j * 16 + l16 < last_n ? j * 16 + l16 : last_n;
            offB[j] = packed ? (uint32_t)weight_code_offset(row, quad * 16, g.ldb) : (uint32_t)row * (uint32_t)g.ldb + quad * 16;
        }
    }

    const int KT = (int)((g.K + 63) / 64);
    const int n = wave < KT ? (KT - wave + NW - 1) / NW : 0;  // steps of this wavefront
    i32x4 fa[D][MB], fb[D][NB], acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = (i32x4){0, 0, 0, 0};

    // CHECKED: the step may be the last, ragged one or lie past the end: chunks of A past the contraction are zeros, so the
    // product of whatever B holds there (packing) vanishes, and rows of B past it are not touched
    auto fetch = [&](int i, i32x4 (&a)[MB], i32x4 (&b)[NB], auto checked) {
        constexpr bool CHECKED = decltype(checked)::value;
        const int8_t* const zero = reinterpret_cast<const int8_t*>(kZeroChunk);
        const int64_t kt = wave + i * NW, k0 = kt * 64;
        const int8_t* const pb = tileB + kt * stepB;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int8_t* src = pb + offB[q];
            if (CHECKED && k0 + (BT ? 2 * (q * 8 + (lane >> 3)) : 0) >= g.K) src = zero;
            b[q] = *reinterpret_cast<const i32x4*>(src);
        }
        const int8_t* const pa = tileA + k0;
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int8_t* src = pa + offA[q];
            if (CHECKED && k0 + quad * 16 >= g.K) src = zero;
            a[q] = *reinterpret_cast<const i32x4*>(src);
        }
    };
    // BT: the 64 x 64 bytes of a step go through this wavefront's 4 KB of LDS: 16-byte chunk c of contraction row k sits in
    // slot 4 k + (c ^ x(k)), x = bits 2 and 4 of k, which spreads the 16 rows that half a wavefront's transposing read
    // touches over all banks.  The LDS serves a wavefront's accesses in order: no wait between the writes and the reads.
    lds_i8* const tr = lds + wave * 4096;
    auto swz = [](int k) { return ((k >> 2) & 1) | ((k >> 3) & 2); };
    auto multiply = [&](const i32x4 (&a)[MB], const i32x4 (&b)[NB]) {
        i32x4 w[NB];
        if constexpr (BT) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int k = 2 * (q * 8 + (lane >> 3)) + ((lane >> 2) & 1), c = lane & 3;
                *(lds_i32x4*)(tr + k * 64 + (c ^ swz(k)) * 16) = b[q];
            }
            const int jj = l16 >> 1, piece = l16 & 1;          // lane mapping of the transposing read: see BtStage
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int k = quad * 16 + jj;
                const i32x2 lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(tr + k * 64 + (j ^ swz(k)) * 16 + piece * 8));
                const i32x2 hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                    (lds_i32x2*)(tr + (k + 8) * 64 + (j ^ swz(k + 8)) * 16 + piece * 8));
                w[j] = (i32x4){lo[0], lo[1], hi[0], hi[1]};
            }
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j) w[j] = b[j];
        }
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[j], a[i], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, fa[d], fb[d], std::true_type{});
    int i = 0;
    for (; i + 2 * D < n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(fa[d], fb[d]);
            fetch(i + D + d, fa[d], fb[d], std::false_type{});
        }
    }
    for (; i + D < n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(fa[d], fb[d]);
            fetch(i + D + d, fa[d], fb[d], std::true_type{});
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (i + d < n) multiply(fa[d], fb[d]);                // (uniform over the wavefront)

    const bool dump = g.acc1 != nullptr;
    const int nk = g.K2 / 64;
    const int planes8 = g.r / 8;                              // 8-column chunks of r per plane of T
#pragma unroll
    for (int rd = 0; rd < C::ROUNDS; ++rd) {
        const int blk = rd * C::PER_ROUND + wave;             // the block this wavefront finishes
        const int bi = blk / NB, bj = blk % NB;
        const bool mine = wave < C::PER_ROUND && m0 + bi * 16 < g.M && n0 + bj * 16 < g.N;
        const int row = bi * 16 + l16 < last_m ? bi * 16 + l16 : last_m;
        // its epilogue operands: first slice of the outlier product, 32 columns' worth of the low-rank one, scales
        i32x4 a2 = {}, b2 = {}, t0 = {}, u0 = {};
        float rs = 1.0f;
        float cs[4] = {1.0f, 1.0f, 1.0f, 1.0f}, cs2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const int8_t* const pa2 = g.A2 + (m0 + row) * g.K2 + quad * 16;
        const int8_t* const pb2 = g.B2 + (n0 + bj * 16 + l16) * g.K2 + quad * 16;
        // the low-rank contraction is the four planes (hi and lo of both parts) one after the other, 8 columns per lane
        auto chunk_t = [&](int q) {
            const int plane = q / planes8, col = (q % planes8) * 8;
            const uint16_t* base = (plane & 1) ? g.T_lo : g.T_hi;
            return *reinterpret_cast<const i32x4*>(base + ((int64_t)(plane >> 1) * g.M + m0 + row) * g.r + col);
        };
        auto chunk_l = [&](int q) {
            return *reinterpret_cast<const i32x4*>(g.L + (n0 + bj * 16 + l16) * g.r + (q % planes8) * 8);
        };
        if (mine && !dump) {
            if (nk > 0) {
                a2 = *reinterpret_cast<const i32x4*>(pa2);
                b2 = *reinterpret_cast<const i32x4*>(pb2);
            }
            if (g.r > 0) {
                t0 = chunk_t(quad);
                u0 = chunk_l(quad);
            }
            rs = g.row_scale[m0 + row];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (g.col_scale) cs[v] = g.col_scale[n0 + bj * 16 + quad * 4 + v];
                if (nk > 0) cs2[v] = g.col_scale2[n0 + bj * 16 + quad * 4 + v];
            }
        }
        if (rd > 0 || BT) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();                     // the exchange area is free
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int b = 0; b < C::PER_ROUND; ++b) {
            const int bb = rd * C::PER_ROUND + b;
            *(lds_i32x4*)(lds + (wave * C::PER_ROUND + b) * 1024 + lane * 16) = acc[bb / NB][bb % NB];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (!mine) continue;
        i32x4 sum = {};
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += *(const lds_i32x4*)(lds + (w * C::PER_ROUND + wave) * 1024 + lane * 16);

        i32x4 acc2 = {};
        const int64_t orow = m0 + bi * 16 + l16, ocol = n0 + bj * 16 + quad * 4;
        if (nk > 0) {
            if (dump) {
                a2 = *reinterpret_cast<const i32x4*>(pa2);
                b2 = *reinterpret_cast<const i32x4*>(pb2);
            }
            acc2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(b2, a2, acc2, 0, 0, 0);
            for (int kk = 1; kk < nk; ++kk)
                acc2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const i32x4*>(pb2 + kk * 64),
                                                             *reinterpret_cast<const i32x4*>(pa2 + kk * 64), acc2, 0, 0, 0);
        }
        if (dump) {
            if (orow < g.M) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    g.acc1[orow * g.N + ocol + v] = sum[v];
                    if (g.acc2) g.acc2[orow * g.N + ocol + v] = acc2[v];
                }
            }
            continue;
        }
        f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
        if (g.r > 0) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u0), __builtin_bit_cast(bf16x8, t0), c, 0, 0, 0);
            for (int q = 4; q < 2 * kLoraParts * planes8; q += 4)
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, chunk_l(q + quad)),
                                                            __builtin_bit_cast(bf16x8, chunk_t(q + quad)), c, 0, 0, 0);
        }
        if (orow >= g.M) continue;
        float* const out = g.C + orow * g.ldc + ocol;
        if (g.accumulate) {
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] += out[v];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            c[v] = __builtin_fmaf(rs, __builtin_fmaf((float)sum[v], cs[v], (float)acc2[v] * cs2[v]), c[v]);
        if (g.C16) {
            uint32_t h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t u = __float_as_uint(c[v]);
                h[v] = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
            }
            *reinterpret_cast<i32x2*>(g.C16 + orow * g.ldc + ocol) = (i32x2){(int)(h[0] | (h[1] << 16)), (int)(h[2] | (h[3] << 16))};
        } else if (g.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(g.C) & 15u) == 0) {
            *reinterpret_cast<f32x4*>(out) = c;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) out[v] = c[v];
        }
    }
}

template <int MB, int NB, int NW, int D, bool BT>
static hipError_t launch_rows(const GemmArgs& g, hipStream_t stream) {
    using C = RowsCfg<MB, NB, NW, D, BT>;
    const int tiles_m = (int)((g.M + C::BM - 1) / C::BM), tiles_n = (int)((g.N + C::BN - 1) / C::BN);
    TileMap tm = make_tile_map(tiles_m, tiles_n, C::BM, C::BN, 1);
    while ((tm.rm + tm.gm - 1) / tm.gm > 65535) tm.gm *= 2;
    if (tm.rn > 65535) return hipErrorInvalidValue;
    const dim3 grid(8 * (unsigned)tm.gm, (unsigned)tm.rn, (unsigned)((tm.rm + tm.gm - 1) / tm.gm));
    auto k = gemm_i8_rows_kernel<MB, NB, NW, D, BT>;
    hipLaunchKernelGGL(k, grid, dim3(C::NT), C::LDS_BYTES, stream, g, tm);
    return hipGetLastError();
}

hipError_t launch_gemm_rows(const GemmArgs& g, int shape, hipStream_t stream) {
    if (g.b_layout == kPackedKN) {
        switch (shape) {
            case kRows16x64: return launch_rows<1, 4, 16, 2, true>(g, stream);
            case kRows32x64: return launch_rows<2, 4, 4, 3, true>(g, stream);
        }
    } else {
        switch (shape) {
            case kRows16x16: return launch_rows<1, 1, 8, 4, false>(g, stream);
            case kRows32x32: return launch_rows<2, 2, 4, 4, false>(g, stream);
            case kRows32x64: return launch_rows<2, 4, 8, 3, false>(g, stream);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace quaff
