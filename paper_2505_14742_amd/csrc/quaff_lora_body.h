// Device code of the LoRA down-projection, shared by its stand-alone launch and by the launch that runs it next to
// the quantizer (see quaff_lora.hip for the description).
#pragma once
#include "quaff_internal.h"

namespace quaff {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kLoraWaves = 16;
// 64 columns of the factor (two steps) go through a wavefront's piece of LDS, so that they are fetched as whole lines and the next ones
// are requested before these are multiplied.  [c x r]: as they are, rows of `row` bytes with `pad` more after every 16, back
// through the transposing read ds_read_b64_tr_b16; the four rows that sixteen lanes read lie in different banks (rank 64: the
// 16-byte chunks of rows 2 and 3 of every four trade places two by two).  [r x c]: r rows of 128 bytes, chunk ch of row p in slot
// ch ^ ((p >> 1) & 7).  `depth` pairs of steps are in flight.  The sums over the wavefronts use the same memory afterwards: at
// rank 16 the 40 KB then fit beside a workgroup of the input-gradient product.
// Launches, us, factor fetched fragment by fragment ([c x r] from rank 32 on through a copy transposed by a launch of 4.8 us) / so: abs-max
// and down-projection at rank 64, 4096 x 4096 20.8 / 16.8; X A at rank 64, 4096 x 4096 18.1 / 13.8, at rank 16, 2048 x 8192 18.6 / 13.8;
// backward quantizer and down-projection at rank 64, 4096 x 11008 61.7 / 55.0, at rank 32, 1003 x 2064 10.7 / 7.4.
template <int R16, bool L_RC> struct LoraRows {
    static constexpr int row = R16 * 32, pad = R16 == 1 ? 128 : R16 == 4 ? 0 : 32, block = 16 * row + pad;
    static constexpr int bytes = L_RC ? R16 * 16 * 128 : 4 * block;
    static constexpr int depth = R16 == 1 ? 2 : 1;
};
// LDS of lora_down_body
template <int R16, bool L_RC> constexpr int lora_lds_bytes() {
    return kLoraWaves * (LoraRows<R16, L_RC>::bytes > R16 * 1024 ? LoraRows<R16, L_RC>::bytes : R16 * 1024);
}
// Row groups of 16 rows per workgroup.  From rank 48 on a workgroup takes 32 rows: every workgroup fetches its share of
// L (c x r against 16 x c of rows: four times the rows' bytes at rank 64), and its 128 registers per lane leave room
// for one 16-wavefront workgroup per compute unit only, so 16-row workgroups would also need two rounds at 4096 rows.
// Measured at rank 64, 4096 rows: abs-max + down-projection launch 43 -> 30 us at 4096 columns, 86 -> 64 us at 11008;
// backward quantizer + down-projection launch 44 -> 30 us and 96 -> 80 us.
constexpr int lora_row_groups(int R16) { return R16 >= 3 ? 2 : 1; }
inline int lora_rows_per_block(int r) { return 16 * lora_row_groups(r / 16); }

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// R16 = r / 16 column blocks of T.  L_RC: L is [r x c] (contraction-contiguous) else [c x r].  RG = row groups of 16 rows.
// Work of one workgroup (64 * kLoraWaves threads): `bx` < row_blocks is its block of 16 RG rows and `by` its part of the
// contraction range; workgroups bx >= row_blocks (nbx in all, by = 0 only) write the transposed copy.
template <int R16, bool L_RC, int RG = 1, int DEPTH = LoraRows<R16, L_RC>::depth>
__device__ __forceinline__ void lora_down_body(char* lora_lds, int bx, int by, int nbx, const uint16_t* __restrict__ X, int64_t t, int c,
                                               int64_t ldx, const uint16_t* __restrict__ L, float scale,
                                               uint16_t* __restrict__ T_hi, uint16_t* __restrict__ T_lo, int row_blocks,
                                               const uint16_t* __restrict__ tr_src, uint16_t* __restrict__ tr_dst,
                                               int64_t tr_rows, int64_t tr_cols) {
    constexpr int r = R16 * 16;
    constexpr int NT = 64 * kLoraWaves;
    using Rows = LoraRows<R16, L_RC>;
    if (bx >= row_blocks) {
        if (by != 0) return;
        // transposed copy: dst [cols x rows] <- src [rows x cols]
        const uint32_t total = (uint32_t)(tr_rows * tr_cols), rows = (uint32_t)tr_rows;     // (at most 64 x 2^20)
        for (uint32_t e = (uint32_t)(bx - row_blocks) * NT + threadIdx.x; e < total; e += (uint32_t)(nbx - row_blocks) * NT)
            tr_dst[e] = tr_src[(int64_t)(e % rows) * tr_cols + e / rows];
        return;
    }
    float (*red)[R16][64][4] = reinterpret_cast<float (*)[R16][64][4]>(lora_lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, g = lane >> 4;
    bool live[RG];
    const uint16_t* xrow[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        const int64_t row = ((int64_t)bx * RG + rg) * 16 + m;
        live[rg] = row < t;
        xrow[rg] = X + (live[rg] ? row : 0) * ldx;
    }

    f32x4 acc[RG][R16];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int b = 0; b < R16; ++b) acc[rg][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // each wavefront owns one contiguous slice of the contraction range (kw columns), walked in 32-column steps
    // this workgroup's part of the contraction range, then this wavefront's slice of it
    // (multiples of 64 columns = 128 bytes, so that a pair of steps reads whole cache lines, see below)
    const int cp = ((c + kLoraParts * 64 - 1) / (kLoraParts * 64)) * 64;
    const int cbeg = by * cp, cend = cbeg + cp < c ? cbeg + cp : c;
    const int kw = ((cend - cbeg + kLoraWaves * 64 - 1) / (kLoraWaves * 64)) * 64;
    const int kbeg = cbeg + wave * kw, kend = kbeg + kw < cend ? kbeg + kw : cend;
    T_hi += (int64_t)by * t * r;
    T_lo += (int64_t)by * t * r;
    // Two consecutive steps share 64 columns: lane group g takes columns 16 g .. 16 g + 7 in the even step and 16 g + 8 .. 16 g + 15
    // in the odd one (any assignment of contraction indices to MFMA slots is valid as long as both operands use it), so the four
    // groups of a row read one whole 128-byte line per step pair instead of two half lines.
    auto mfmas = [&](const u32x4 (&x)[RG], const u32x4 (&l)[R16]) {
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
#pragma unroll
            for (int b = 0; b < R16; ++b)
                acc[rg][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[rg]), __builtin_bit_cast(bf16x8, l[b]),
                                                                     acc[rg][b], 0, 0, 0);
    };
    typedef short v4s __attribute__((ext_vector_type(4)));
    typedef short v8s __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) v4s lds_v4s;
    constexpr int D = DEPTH, CPR = L_RC ? 8 : r / 8;      // 16-byte chunks per row
    char* const mine = lora_lds + wave * Rows::bytes;
    auto at = [&](int kk, int chunk) {                           // row kk of the pair's 64 (L_RC: of r)
        if (L_RC) return kk * 128 + (chunk ^ ((kk >> 1) & 7)) * 16;
        return (kk >> 4) * Rows::block + (kk & 15) * Rows::row + (R16 == 4 ? chunk ^ (((kk >> 1) & 1) * 2) : chunk) * 16;
    };
    const int pairs = kend > kbeg ? (kend - kbeg + 63) / 64 : 0;
    u32x4 xa[D][2][RG], lb[D][2 * R16];
    auto load = [&](int p, int slot) {
        const int k0 = kbeg + p * 64, k = k0 + g * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg)
                xa[slot][h][rg] = *reinterpret_cast<const u32x4*>(xrow[rg] + (k < kend ? k + h * 8 : c - 8));
#pragma unroll
        for (int i = 0; i < 2 * R16; ++i) {
            const int id = i * 64 + lane, kr = k0 + id / CPR, kc = k0 + (id % CPR) * 8;
            if (L_RC)
                lb[slot][i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(L) +
                                                              (uint32_t)((id / CPR) * c + (kc < c ? kc : c - 8)) * 2u);
            else lb[slot][i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(L) +
                                                          (uint32_t)((kr < c ? kr : c - 1) * (2 * r) + (id % CPR) * 16));
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < pairs) load(d, d);
    for (int p0 = 0; p0 < pairs; p0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int p = p0 + d;
            if (p >= pairs) break;                               // (uniform over the wavefront, whose LDS operations run in order)
#pragma unroll
            for (int i = 0; i < 2 * R16; ++i) {
                const int id = i * 64 + lane;
                *reinterpret_cast<u32x4*>(mine + at(id / CPR, id % CPR)) = lb[d][i];
            }
            u32x4 x[2][RG];                                      // (a step past the end meets zeros)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int rg = 0; rg < RG; ++rg)
                    x[h][rg] = live[rg] && kbeg + p * 64 + g * 16 < kend ? xa[d][h][rg] : (u32x4){0, 0, 0, 0};
            if (p + D < pairs) load(p + D, d);
            // lane (m, g): rank 16 b + m, columns 16 g .. (even step), 16 g + 8 .. (odd); lane m of a group of sixteen addresses
            // column m / 4 of the four it wants, ranks 4 (m % 4) .. + 3, and receives rank m of all four
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 l[R16];
#pragma unroll
                for (int b = 0; b < R16; ++b) {
                    if constexpr (L_RC) {
                        l[b] = *reinterpret_cast<const u32x4*>(mine + at(b * 16 + m, 2 * g + h));
                        continue;
                    }
                    auto four = [&](int col0) {
                        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_v4s*)(mine + at(g * 16 + col0 + (m >> 2), b * 2 + ((m & 3) >> 1)) + (m & 1) * 8));
                    };
                    const v4s f0 = four(h * 8), f1 = four(h * 8 + 4);
                    l[b] = __builtin_bit_cast(u32x4, (v8s){f0[0], f0[1], f0[2], f0[3], f1[0], f1[1], f1[2], f1[3]});
                }
                mfmas(x[h], l);
            }
        }
    }
    __syncthreads();                                                 // (the sums below take the place of the slices)
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        if (rg > 0) __syncthreads();               // the sums over the previous row group have been read
#pragma unroll
        for (int b = 0; b < R16; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][b][lane][v] = acc[rg][b][v];
        __syncthreads();
        // fixed-order sum over the wavefronts; element v of lane (m, g) is T[row0 + 4 g + v][16 b + m]
        for (int e = threadIdx.x; e < R16 * 64 * 4; e += NT) {
            int v = e & 3, ln = (e >> 2) & 63, b = e >> 8;
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < kLoraWaves; ++w) s += red[w][b][ln][v];
            s = s * scale;
            int64_t orow = ((int64_t)bx * RG + rg) * 16 + (ln >> 4) * 4 + v;
            if (orow < t) {
                uint32_t hi = f32_to_bf16_rne(s);
                float rest = s - __uint_as_float(hi << 16);
                T_hi[orow * r + b * 16 + (ln & 15)] = (uint16_t)hi;
                T_lo[orow * r + b * 16 + (ln & 15)] = (uint16_t)f32_to_bf16_rne(rest);
            }
        }
    }
}

}  // namespace quaff
