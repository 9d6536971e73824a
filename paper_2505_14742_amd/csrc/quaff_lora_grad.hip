// LoRA weight gradients of the adapter branch Y_l = scale (X A) B (rank r; the paper's App. "Model and experimental
// settings" puts LoRA on every linear layer, the frozen quantized weight gets no gradient):
//     dA = scale X^T (dY B^T)   [c_in x r]          dB = scale (X A)^T dY   [r x c_out]
// Both are one skinny product  G[p, j] = sum_i P[i, p] Q[i, j]  that contracts over the t tokens:
//     dB:  P = scale X A   (the forward down-projection),  Q = dY
//     dA:  P = scale dY B^T (the backward down-projection), Q = X,  result stored transposed.
// HBM-bound: Q is read once.  bf16 MFMA 16x16x32 with fp32 accumulation.  Both operands have the tokens on the slow
// axis while the MFMA wants them contiguous per lane, so 64-token tiles of both are staged row-major in LDS (two
// buffers used in turn, one barrier per tile, the next tile's global loads in flight while this one is multiplied) and
// a lane gets its eight tokens by two transposing reads.  P arrives as the hi/lo bf16 parts the down-projection kernel
// writes (one pair per half of its contraction range) and is folded to one hi/lo pair while it is staged.  Both
// products of a layer run in one launch.  The token range is cut into slabs over workgroups; the slabs' partial
// results are summed in a fixed order by a second launch that fills the chip, so the result is deterministic.
// (Measured and dropped: the sum done inside the product launch by whichever workgroup of a column chunk finishes
// last, found with a ticket counter.  The sixteen partial results per element have to be fetched past the caches
// by a few workgroups at the tail of the launch; both Phi-3 attention projections took 0.129 ms against 0.079 ms.)
#include "quaff_internal.h"

namespace quaff {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kGradCols = 128;       // columns of Q per workgroup of four wavefronts (two 16-column MFMA blocks each)
constexpr int kGradTokens = 64;      // tokens per staged tile

__device__ __forceinline__ uint32_t grad_f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

void lora_grad_plan(int64_t t, int64_t c, int* nslab, int* rows_per_slab) {
    const int64_t tiles = (t + kGradTokens - 1) / kGradTokens;
    const int64_t chunks = (c + kGradCols - 1) / kGradCols;
    int64_t want = (512 + chunks - 1) / chunks;            // about two workgroups per compute unit
    // at most eight slabs: the partial results are written and read once more, and the launch that sums them gets
    // longer with every slab (measured at 2048 tokens: 16 slabs 41 / 31 us per call for the two Phi-3 attention
    // projections, 8 slabs 36 / 29 us, 4 slabs 38 / 31 us)
    if (want > 8) want = 8;
    // up to 256 tokens one slab, written straight to the result: the launch that sums them costs more than the tiles
    if (tiles <= 4) want = 1;
    if (want > tiles) want = tiles;
    const int64_t rows = ((tiles + want - 1) / want) * kGradTokens;
    *rows_per_slab = (int)rows;
    *nslab = (int)((tiles * kGradTokens + rows - 1) / rows);
}

// partial[slab][p][j] = sum over the slab's tokens i of P[i, p] Q[i, j];  P = the sum of the kLoraParts hi/lo pairs of T.
// One of the two products of a launch (blockIdx.z selects it).
struct GradProblem {
    const uint16_t* Q; int64_t ldq; int c;
    const uint16_t* T_hi; const uint16_t* T_lo;       // [kLoraParts][t][r]
    int rows_per_slab, nslab, chunks;
    float* partial; int transposed;                   // [nslab][r][c], or [nslab][c][r] if transposed
    float* out;                                       // their sum (nslab = 1: partial = out)
};
struct GradPair { GradProblem p[2]; };

// The transposing LDS read: in each group of 16 lanes, lane i receives 16-bit element i % 4 of the 8-byte pieces addressed by
// lanes i / 4 + 4 j, j = 0..3; lane a of a group therefore addresses row a / 4 of four, elements 4 (a % 4) .. + 3 of 16.
typedef short grad_v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) grad_v4s lds_grad_v4s;

// LDS position of 32-byte pair `pair` (16 columns) of token row `row` in a Q tile of NPAIR pairs per row: the pairs of the
// eight rows that half a wavefront's transposing read touches (four rows, and four rows 8 further on) lie in different banks.
template <int NPAIR>
__device__ __forceinline__ int grad_q_offset(int row, int pair) {
    return row * NPAIR * 32 + (pair ^ (row & 3) ^ ((row >> 1) & 4)) * 32;
}

// NW wavefronts, 32 columns each.  (Gathering the operands with 2-byte LDS reads takes ten times as many instructions at rank
// 64 as the MFMAs they feed.  The whole call at 4096 x (4096, 11008) and rank 64: 99 us, with gathered operands and slabs that lie
// across the result 147; 512 x (3072, 3072) at rank 16: 15.7 and 18.5.)
template <int R16, int NW>
__global__ void __launch_bounds__(NW * 64)
lora_grad_kernel(GradPair pair, int64_t t) {
    constexpr int r = R16 * 16, NT = NW * 64, COLS = NW * 32;
    constexpr int PSTR = r * 2 == 128 ? 160 : r * 2;      // bytes per token of a staged P tile (four rows in disjoint banks)
    constexpr int QTILE = kGradTokens * COLS * 2, PTILE = kGradTokens * PSTR;
    constexpr int PV = kGradTokens * r / 8;               // 16-byte vectors of a P tile
    constexpr int PJ = (PV + NT - 1) / NT;                // ... per thread
    const GradProblem& pb = pair.p[blockIdx.z];
    if ((int)blockIdx.x >= pb.chunks || (int)blockIdx.y >= pb.nslab) return;
    const uint16_t* __restrict__ Q = pb.Q;
    const int64_t ldq = pb.ldq;
    const int c = pb.c;
    const uint16_t* __restrict__ T_hi = pb.T_hi;
    const uint16_t* __restrict__ T_lo = pb.T_lo;
    extern __shared__ __attribute__((aligned(16))) uint8_t grad_lds[];   // Q tiles [2], then P tiles [2][hi, lo]
    uint8_t* const qt = grad_lds;
    uint8_t* const pt = grad_lds + 2 * QTILE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int c0 = blockIdx.x * COLS;
    const int64_t t_pad = (t + kGradTokens - 1) / kGradTokens * kGradTokens;
    const int64_t i_begin = (int64_t)blockIdx.y * pb.rows_per_slab;
    const int64_t i_end = i_begin + pb.rows_per_slab < t_pad ? i_begin + pb.rows_per_slab : t_pad;

    // loaders.  Q: 64 rows x COLS columns, four 16-byte vectors per thread (rows tid / (COLS / 8) + 16 h).
    // P: token tok, rank indices p0 .. p0 + 7 of each of the four arrays (hi / lo of the two contraction parts).
    constexpr int QV = COLS / 8;
    const int ld_row = tid / QV;
    int ld_col = c0 + (tid % QV) * 8;
    if (ld_col > c - 8) ld_col = c - 8;        // columns past the edge repeat valid data and are never stored
    struct TileRegs { u32x4 q[4]; u32x4 p[PJ][2 * kLoraParts]; };
    auto load_tile = [&](int64_t i0, TileRegs& tr) {
        u32x4 (&qreg)[4] = tr.q;
        u32x4 (&preg)[PJ][2 * kLoraParts] = tr.p;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            int64_t row = i0 + ld_row + 16 * h;
            if (row > t - 1) row = t - 1;      // tokens past the end repeat the last one; P is zero there
            qreg[h] = *reinterpret_cast<const u32x4*>(Q + row * ldq + ld_col);
        }
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
            const int v = tid + NT * j;
            const int tok = v / (r / 8), p0 = (v % (r / 8)) * 8;
            const int64_t i = i0 + tok;
#pragma unroll
            for (int part = 0; part < kLoraParts; ++part) {
                preg[j][2 * part] = preg[j][2 * part + 1] = (u32x4){0, 0, 0, 0};
                if (v < PV && i < t) {
                    const int64_t o = ((int64_t)part * t + i) * r + p0;
                    preg[j][2 * part] = *reinterpret_cast<const u32x4*>(T_hi + o);
                    preg[j][2 * part + 1] = *reinterpret_cast<const u32x4*>(T_lo + o);
                }
            }
        }
    };
    auto stage_tile = [&](int buf, const TileRegs& tr) {
        const u32x4 (&qreg)[4] = tr.q;
        const u32x4 (&preg)[PJ][2 * kLoraParts] = tr.p;
#pragma unroll
        for (int h = 0; h < 4; ++h)
            *reinterpret_cast<u32x4*>(qt + buf * QTILE + grad_q_offset<COLS / 16>(ld_row + 16 * h, (tid % QV) >> 1) + (tid & 1) * 16) =
                qreg[h];
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
            const int v = tid + NT * j;
            if (v >= PV) continue;
            const int tok = v / (r / 8), p0 = (v % (r / 8)) * 8;
            uint32_t hi2[4], lo2[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t hpair = 0, lpair = 0;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    float sum = 0.0f;          // the parts in their order, each as hi + lo
#pragma unroll
                    for (int part = 0; part < kLoraParts; ++part) {
                        const uint32_t hw = preg[j][2 * part][w], lw = preg[j][2 * part + 1][w];
                        const float hf = __uint_as_float(half ? (hw & 0xFFFF0000u) : (hw << 16));
                        const float lf = __uint_as_float(half ? (lw & 0xFFFF0000u) : (lw << 16));
                        sum += hf + lf;
                    }
                    const uint32_t hi = grad_f32_to_bf16_rne(sum);
                    const uint32_t lo = grad_f32_to_bf16_rne(sum - __uint_as_float(hi << 16));
                    hpair |= hi << (16 * half);
                    lpair |= lo << (16 * half);
                }
                hi2[w] = hpair;
                lo2[w] = lpair;
            }
            *reinterpret_cast<u32x4*>(pt + (buf * 2 + 0) * PTILE + tok * PSTR + p0 * 2) = (u32x4){hi2[0], hi2[1], hi2[2], hi2[3]};
            *reinterpret_cast<u32x4*>(pt + (buf * 2 + 1) * PTILE + tok * PSTR + p0 * 2) = (u32x4){lo2[0], lo2[1], lo2[2], lo2[3]};
        }
    };
    auto join8 = [](const uint8_t* first4, const uint8_t* last4) {
        const grad_v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_grad_v4s*)first4);
        const grad_v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_grad_v4s*)last4);
        return __builtin_bit_cast(u32x4, (short __attribute__((ext_vector_type(8)))){a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
    };

    f32x4 acc[R16][2];
#pragma unroll
    for (int b = 0; b < R16; ++b)
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[b][f] = (f32x4){0.f, 0.f, 0.f, 0.f};

    auto multiply_tile = [&](int buf) {
#pragma unroll
        for (int sub = 0; sub < kGradTokens / 32; ++sub) {
            const int row = sub * 32 + g * 8 + (n >> 2), in = (n & 3) * 8;       // this lane's row of the first four tokens
            u32x4 ah[R16], al[R16];
#pragma unroll
            for (int b = 0; b < R16; ++b) {
                const uint8_t* ph = pt + (buf * 2 + 0) * PTILE + row * PSTR + b * 32 + in;
                ah[b] = join8(ph, ph + 4 * PSTR);
                al[b] = join8(ph + PTILE, ph + PTILE + 4 * PSTR);
            }
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                // second operand: eight tokens of column c0 + 16 (2 wave + f) + n
                const uint8_t* q0 = qt + buf * QTILE + in;
                const u32x4 q = join8(q0 + grad_q_offset<COLS / 16>(row, wave * 2 + f), q0 + grad_q_offset<COLS / 16>(row + 4, wave * 2 + f));
#pragma unroll
                for (int b = 0; b < R16; ++b) {
                    acc[b][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ah[b]),
                                                                        __builtin_bit_cast(bf16x8, q), acc[b][f], 0, 0, 0);
                    acc[b][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, al[b]),
                                                                        __builtin_bit_cast(bf16x8, q), acc[b][f], 0, 0, 0);
                }
            }
        }
    };
    // Two tiles are in flight from global memory at any time (two register sets used in turn; the loop body covers
    // two tiles so that which set a tile uses is fixed at compile time), a third is being multiplied out of LDS.
    // One barrier per tile: the barrier of the next tile separates this tile's gathers from the stores that reuse
    // its LDS buffer two tiles on.
    TileRegs ra, rb;
    load_tile(i_begin, ra);
    if (i_begin + kGradTokens < i_end) load_tile(i_begin + kGradTokens, rb);
    for (int64_t i0 = i_begin; i0 < i_end; i0 += 2 * kGradTokens) {
        stage_tile(0, ra);
        __syncthreads();
        if (i0 + 2 * kGradTokens < i_end) load_tile(i0 + 2 * kGradTokens, ra);
        multiply_tile(0);
        if (i0 + kGradTokens < i_end) {
            stage_tile(1, rb);
            __syncthreads();
            if (i0 + 3 * kGradTokens < i_end) load_tile(i0 + 3 * kGradTokens, rb);
            multiply_tile(1);
        }
    }
    // element v of lane (n, g) is G[16 b + 4 g + v][c0 + 16 (2 wave + f) + n]
    float* out = pb.partial + (int64_t)blockIdx.y * r * c;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        const int col = c0 + (wave * 2 + f) * 16 + n;
        if (col >= c) continue;
#pragma unroll
        for (int b = 0; b < R16; ++b) {
            if (pb.transposed) {
#pragma unroll
                for (int v = 0; v < 4; ++v) out[(int64_t)col * r + b * 16 + g * 4 + v] = acc[b][f][v];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) out[(int64_t)(b * 16 + g * 4 + v) * c + col] = acc[b][f][v];
            }
        }
    }
}

// out = sum over slabs (fixed order) of partial[slab], four elements per thread.  (The partial results lie as the result does:
// with dA's slabs in the other order, read across, this launch took 20 us at 4096 x 4096 and rank 64.)
__global__ void __launch_bounds__(256)
lora_grad_reduce_kernel(GradPair pair, int r) {
    const GradProblem& pb = pair.p[blockIdx.y];
    const float* __restrict__ partial = pb.partial;
    float* __restrict__ out = pb.out;
    const int nslab = pb.nslab;
    if (nslab == 1) return;
    const int64_t total = (int64_t)r * pb.c;               // a multiple of 256
    for (int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; e < total; e += (int64_t)gridDim.x * 1024) {
        f32x4 v[8], s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) v[sl] = *reinterpret_cast<const f32x4*>(partial + (sl < nslab ? sl : 0) * total + e);
#pragma unroll
        for (int sl = 0; sl < 8; ++sl)
            if (sl < nslab) s += v[sl];
#pragma unroll
        for (int u = 0; u < 4; ++u) out[e + u] = s[u];
    }
}

size_t lora_grad_lds_bytes(int32_t r, int cols) {
    return 2 * (size_t)kGradTokens * cols * 2 + 4 * (size_t)kGradTokens * (r * 2 == 128 ? 160 : r * 2);
}

// Both gradient products of a layer in one launch:
//   dA^T [r x c_in] = P1^T X (stored transposed as dA [c_in x r]),   dB [r x c_out] = P2^T dY
// with P1 = T1 (the down-projection of dY) and P2 = T2 (the down-projection of X), each given as the hi / lo parts
// [kLoraParts x t x r] that launch_lora_down writes.
hipError_t launch_lora_grad_pair(const uint16_t* X, int64_t ldx, int64_t c_in, const uint16_t* T1_hi,
                                 const uint16_t* T1_lo, float* partial_a, float* dA, const uint16_t* dY, int64_t lddy,
                                 int64_t c_out, const uint16_t* T2_hi, const uint16_t* T2_lo, float* partial_b,
                                 float* dB, int64_t t, int32_t r, hipStream_t stream) {
    ProfScope prof(K_LORA_GRAD, stream);
    GradPair pair;
    // From rank 32 on a workgroup takes 256 columns: the tokens' P (512 bytes a token at rank 64, against 256 of Q per 128
    // columns) is fetched and folded half as often (4096 x (4096, 11008), rank 64: whole call 105 against 99 us; rank 16: level).
    const bool wide = r >= 32;
    const int cols = wide ? 2 * kGradCols : kGradCols;
    auto fill = [&](GradProblem& p, const uint16_t* Q, int64_t ldq, int64_t c, const uint16_t* hi, const uint16_t* lo,
                    float* partial, float* out, int transposed) {
        p.Q = Q; p.ldq = ldq; p.c = (int)c; p.T_hi = hi; p.T_lo = lo;
        lora_grad_plan(t, c, &p.nslab, &p.rows_per_slab);
        p.chunks = (int)((c + cols - 1) / cols);
        p.partial = p.nslab == 1 ? out : partial; p.out = out; p.transposed = transposed;
    };
    fill(pair.p[0], X, ldx, c_in, T1_hi, T1_lo, partial_a, dA, 1);
    fill(pair.p[1], dY, lddy, c_out, T2_hi, T2_lo, partial_b, dB, 0);
    const int gx = pair.p[0].chunks > pair.p[1].chunks ? pair.p[0].chunks : pair.p[1].chunks;
    const int gy = pair.p[0].nslab > pair.p[1].nslab ? pair.p[0].nslab : pair.p[1].nslab;
    dim3 grid((unsigned)gx, (unsigned)gy, 2);
    const size_t lds = lora_grad_lds_bytes(r, cols);
#define QUAFF_GRAD(N)                                                                                                 \
    case N: {                                                                                                         \
        auto kern = wide ? lora_grad_kernel<N, 8> : lora_grad_kernel<N, 4>;                                           \
        hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                      \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                    \
        if (ea != hipSuccess) return ea;                                                                              \
        hipLaunchKernelGGL(kern, grid, dim3(wide ? 512 : 256), lds, stream, pair, t);                                 \
    } break;
    switch (r / 16) {
        QUAFF_GRAD(1) QUAFF_GRAD(2) QUAFF_GRAD(3) QUAFF_GRAD(4)
    }
#undef QUAFF_GRAD
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pair.p[0].nslab == 1 && pair.p[1].nslab == 1) return hipSuccess;
    const int64_t cmax = c_in > c_out ? c_in : c_out;
    int64_t blocks = ((int64_t)r * cmax + 1023) / 1024;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(lora_grad_reduce_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, stream, pair, (int)r);
    return hipGetLastError();
}

}  // namespace quaff
