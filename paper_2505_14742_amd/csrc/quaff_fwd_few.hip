// Forward step of a layer in ONE launch, for few rows or few columns (quaff_linear_fwd_step): the outlier-column abs-max (Eq. 8),
// the momentum update (Eq. 7), the requantization of what (Eq. 5, Eq. 9), the scaled per-token quantizer (Eq. 5, Eq. 1), the
// LoRA down-projection and the product with its epilogue (Eq. 9).
//
// Two launches of such a pass - preparation, product - consist of launch, chains of memory round trips and the grid-wide wait
// for the column maxima.  Here a workgroup computes a tile of 16 rows x 16 NB output channels from X itself: it gathers the
// outlier columns of ALL rows (t n values), quantizes its 16 rows and requantizes its channels.  Workgroups of one row of tiles repeat
// the quantizer's work, those of one column the channels', and nobody waits for anybody.  The weight codes, the bulk of the bytes, are
// requested right after the preparation's own operands and travel while it computes.
// The eight wavefronts share the contraction: a wavefront loads, quantizes and multiplies the same 64-column steps.  Lane (m, g)
// holds row m, columns 16 g .. 16 g + 15 of a step, which is at once the layout of whole-line loads, of the down-projection's operand
// and, as 16 codes, of the product's operand in v_mfma_i32_16x16x64_i8: the codes never leave the registers.  Integer partial
// sums meet in LDS, the down-projection's in the order of lora_down_body, so that all results are those of the separate calls.
//
// The new scales may overwrite the old ones only when every workgroup has read them.  A workgroup that has writes its mark (hashed
// from epoch + 1, `epoch` a word of the workspace read before) into a word of its own and looks at all words once at its end;
// whoever finds every mark - the last one to write always does - publishes s, 1 / s, cmax and the new epoch and clears the words.
// Us, two launches / this one: 28 x 256 -> 256 with 2 outliers and rank 16 11.7 / 7.7, 21 x 960 -> 192 with 7 outliers 11.6 / 8.4,
// 7 x 320 -> 512 with rank 16 8.5 / 5.1, 151 x 1536 -> 512 with rank 16 14.5 / 9.7.  What is left is the launch, three round trips and the
// fetch of instructions that run once: the code is kept short (channel steps once per thread, rows of the gather in a loop).
#include "quaff_gemm_dma.h"
#include "quaff_quant_body.h"
#include "quaff_lora_body.h"
#include "quaff_scale_body.h"

namespace quaff {

namespace {
constexpr int kFewRows = 16, kFewWaves = 8, kFewThreads = 64 * kFewWaves;
constexpr int kFewSlices = 16;                 // slices of a part of the down-projection's contraction (lora_down_body's wavefronts)
constexpr int kFewLt = 640;                    // bytes of 16 rows of A in LDS: 16 x 32 + padding
static_assert(kFewSlices == kLoraWaves && kLoraParts == 2, "summation order of lora_down_body");
}  // namespace

struct FwdFewArgs {
    const uint16_t* X; int64_t t; int c; int64_t ldx;
    int n;
    const float* wmax_O; float gamma; float* s_O; float* colscale; float* cmax_out;
    const float* W_O; int c_out; int8_t* what_int; float* delta_what;
    int8_t* Xq; float* delta; int8_t* xq_O;
    const int8_t* Wq; int64_t cpad; const float* delta_w;
    const uint16_t* A; const uint16_t* B; float scale;
    float* Y; int64_t ldy;
    uint64_t* words; uint64_t* epoch;
};

// SPS: 64-column steps of a slice, SL: slices of a wavefront at most, NB: 16-channel blocks of a tile.  (At most 2048 columns: SPS is 1, and all
// steps of A and of the weights are in flight.  Written for that alone the compiler orders the loads differently: 17 x 704 -> 1120 with 38 outliers
// 13.5 -> 15.8 us, 30 x 1536 -> 2432 11.0 -> 11.7.)
template <int SPS, int SL, int NB, bool HAS_LORA>
__global__ void __launch_bounds__(kFewThreads)
fwd_few_kernel(const FwdFewArgs a, const int32_t* __restrict__ O) {
    constexpr int STEPS = SPS * SL, BN = NB * 16;
    // weight steps in flight: what the registers leave beside X (8 a step) and A
    constexpr int PD_ROOM = (150 - 8 * STEPS) / (4 * NB), PD = PD_ROOM < 2 ? 2 : PD_ROOM;
    constexpr int AB = !HAS_LORA || STEPS > 8 ? 2 : STEPS == 6 ? 3 : STEPS < 4 ? STEPS : 4;     // steps of A in flight
    static_assert(!HAS_LORA || STEPS % AB == 0, "whole batches");
    extern __shared__ __attribute__((aligned(16))) char few_lds[];
    float* const cs_copy = reinterpret_cast<float*>(few_lds);                       // column scales [c]
    char* const lt = few_lds + (((size_t)a.c * 4 + 255) & ~(size_t)255);            // per wavefront: a step of A
    // the down-projection's partial sums [32 slices][64 lanes][4], then the product's [wavefront][block][64 lanes][4]
    char* const area = lt + (HAS_LORA ? kFewWaves * 4 * kFewLt : 0);
    __shared__ float rmax[kFewWaves][kFewRows];
    __shared__ uint32_t smax[64];
    __shared__ float snew[64], sm1[64], rinv[64], dw[BN], dwh[BN], rowd[kFewRows];
    __shared__ uint32_t wmaxbits[BN];
    __shared__ __attribute__((aligned(16))) int8_t wcodes[BN][64], xoc[kFewRows][64];
    __shared__ __attribute__((aligned(16))) uint16_t bt[HAS_LORA ? BN : 1][16], tl[HAS_LORA ? 4 : 1][kFewRows][16];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int n = a.n, c = a.c, tiles_n = gridDim.x, tn = blockIdx.x;
    const int64_t row0 = (int64_t)blockIdx.y * kFewRows, row = row0 + m;
    const int n0 = tn * BN, nlive = a.c_out - n0 < BN ? a.c_out - n0 : BN;          // live channels (a multiple of 16)
    const bool live = row < a.t;
    const uint16_t* const xrow = a.X + (live ? row : 0) * a.ldx;

    // ---- the slices of the two parts that hold columns, dealt to the wavefronts in order
    const int cp = ((c + kLoraParts * 64 - 1) / (kLoraParts * 64)) * 64;
    const int len0 = cp < c ? cp : c, len1 = c - len0;
    const int kw0 = ((len0 + kFewSlices * 64 - 1) / (kFewSlices * 64)) * 64, kw1 = ((len1 + kFewSlices * 64 - 1) / (kFewSlices * 64)) * 64;
    const int na0 = (len0 + kw0 - 1) / kw0, na1 = len1 > 0 ? (len1 + kw1 - 1) / kw1 : 0;
    const int per = (na0 + na1 + kFewWaves - 1) / kFewWaves;
    auto slice_of = [&](int j) { return wave * per + j; };
    auto has_slice = [&](int j) { return j < per && slice_of(j) < na0 + na1; };
    auto slice_id = [&](int j) { const int s = slice_of(j); return s < na0 ? s : kFewSlices + s - na0; };
    auto slice_beg = [&](int j) { const int s = slice_of(j); return s < na0 ? s * kw0 : cp + (s - na0) * kw1; };
    auto slice_end = [&](int j) {
        const int s = slice_of(j), e = s < na0 ? (s + 1) * kw0 : cp + (s - na0 + 1) * kw1, lim = s < na0 ? len0 : c;
        return e < lim ? e : lim;
    };
    auto step_col = [&](int u) { return slice_beg(u / SPS) + (u % SPS) * 64; };
    auto step_on = [&](int u) { return has_slice(u / SPS) && step_col(u) < slice_end(u / SPS); };   // uniform over the wavefront

    // ---- global loads, in the order in which they are needed (they return in order)
    int ocol = 0;
    if (lane < n) ocol = O[lane];
    uint64_t epoch = 0;
    float s_prev = 1.0f, wmax_k = 0.0f;
    if (n > 0) {
        epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid < n) {
            s_prev = a.s_O[tid];
            wmax_k = a.wmax_O[tid];
        }
    }
    u32x4 xa[STEPS][2];
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        xa[u][0] = xa[u][1] = (u32x4){0, 0, 0, 0};
        const int k = step_col(u) + g * 16;
        if (step_on(u) && live && k < c) {                      // (c is a multiple of 16)
            xa[u][0] = *reinterpret_cast<const u32x4*>(xrow + k);
            xa[u][1] = *reinterpret_cast<const u32x4*>(xrow + k + 8);
        }
    }
    // outlier columns k = wave + 8 i of all rows, and this tile's rows of columns 8 wave + 4 i + g
    uint32_t cmx[8];
    uint16_t xo[2] = {0, 0};
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) cmx[i] = 0;
        for (int64_t r = 0; r < a.t; r += 64) {
            uint32_t v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = 0;
                if (wave + 8 * i < n && r + lane < a.t)
                    v[i] = a.X[(r + lane) * a.ldx + __builtin_amdgcn_readlane(ocol, wave + 8 * i)];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) cmx[i] = max(cmx[i], v[i] & 0x7FFFu);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = wave * 8 + i * 4 + g, col = __shfl(ocol, k, 64);
            if (k < n && live) xo[i] = a.X[row * a.ldx + col];
        }
    }
    static_assert(2 * kFewSlices * 64 <= 4 * kFewThreads, "columns: a vector of their scales to a thread");
    f32x4 cs_first = {1.f, 1.f, 1.f, 1.f};
    if (tid * 4 < c) cs_first = *reinterpret_cast<const f32x4*>(a.colscale + tid * 4);
    constexpr int WV = 64 * BN / kFewThreads;                   // values of W_O of a thread: element e = (k, channel)
    float w_o[WV];
#pragma unroll
    for (int i = 0; i < WV; ++i) {
        const int e = tid + i * kFewThreads, k = e / BN, jl = e % BN;
        w_o[i] = 0.0f;
        if (k < n && jl < nlive) w_o[i] = a.W_O[(int64_t)k * a.c_out + n0 + jl];
    }
    float dw_first = 0.0f;
    if (tid < nlive) dw_first = a.delta_w[n0 + tid];
    uint16_t b_first[HAS_LORA ? (16 * BN + kFewThreads - 1) / kFewThreads : 1];
    if constexpr (HAS_LORA) {
#pragma unroll
        for (int i = 0; i < (16 * BN + kFewThreads - 1) / kFewThreads; ++i) {
            const int e = tid + i * kFewThreads;
            b_first[i] = 0;
            if (e < 16 * BN && e % BN < nlive) b_first[i] = a.B[(int64_t)(e / BN) * a.c_out + n0 + e % BN];
        }
    }
    u32x4 av[AB][2];
    auto load_a = [&](int u0) {
#pragma unroll
        for (int uu = 0; uu < AB; ++uu)
            if (step_on(u0 + uu)) {
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    int kr = step_col(u0 + uu) + v * 32 + (lane >> 1);         // (a row past the end meets zeros of x)
                    kr = kr < c ? kr : c - 1;
                    av[uu][v] = *reinterpret_cast<const u32x4*>(a.A + (int64_t)kr * 16 + (lane & 1) * 8);
                }
            }
    };
    if constexpr (HAS_LORA) load_a(0);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t off_w[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int ch = j * 16 + m < nlive ? j * 16 + m : nlive - 1;             // (channels past the edge are never stored)
        off_w[j] = (uint32_t)weight_code_offset(ch, g * 16, a.cpad);
    }
    const int8_t* const wtile = a.Wq + (int64_t)n0 * a.cpad;                    // (n0 is even)
    i32x4 fb[PD < STEPS ? PD : STEPS][NB];
    auto fetch_w = [&](int u) {
        if (step_on(u)) {
            const int8_t* const pb = wtile + (int64_t)(step_col(u) >> 6) * 128;
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[u % PD][j] = *reinterpret_cast<const i32x4*>(pb + off_w[j]);
        }
    };
#pragma unroll
    for (int u = 0; u < (PD < STEPS ? PD : STEPS); ++u) fetch_w(u);
    __builtin_amdgcn_sched_barrier(0);

    // ---- column maxima over all rows
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = wave + 8 * i;
            if (k < n) {
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) cmx[i] = max(cmx[i], (uint32_t)__shfl_xor((int)cmx[i], off, 64));
                if (lane == 0) smax[k] = cmx[i] << 16;
            }
        }
    }
    if (tid * 4 < c) *reinterpret_cast<f32x4*>(cs_copy + tid * 4) = cs_first;
    if (tid < BN) {
        dw[tid] = dw_first;
        wmaxbits[tid] = 0u;
    }
    if constexpr (HAS_LORA) {
#pragma unroll
        for (int i = 0; i < (16 * BN + kFewThreads - 1) / kFewThreads; ++i) {
            const int e = tid + i * kFewThreads;
            if (e < 16 * BN) bt[e % BN][e / BN] = b_first[i];
        }
    }
    if (tid < n) snew[tid] = s_prev;           // (the old scales and the epoch have been read when the barrier is passed)
    const uint64_t mark = ((epoch + 1) * 0x9E3779B97F4A7C15ull) | 1ull;
    __syncthreads();
    const int groups = tiles_n * (int)gridDim.y;
    if (n > 0 && tid == kFewThreads - 64)
        __hip_atomic_store(&a.words[(int)blockIdx.y * tiles_n + tn], mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- the new scales; the down-projection's partial sums
    if (tid < n) {
        const float s = momentum_scale(__uint_as_float(smax[tid]), wmax_k, s_prev, a.gamma);
        const float ri = __fdiv_rn(1.0f, s);
        snew[tid] = s;
        sm1[tid] = __fsub_rn(s, 1.0f);
        rinv[tid] = ri;
        cs_copy[ocol] = ri;                    // (tid < 64: lane = tid)
    }
    if constexpr (HAS_LORA) {
        typedef short v4s __attribute__((ext_vector_type(4)));
        typedef short v8s __attribute__((ext_vector_type(8)));
        typedef __attribute__((address_space(3))) v4s lds_v4s;
        char* const mine = lt + wave * 4 * kFewLt;
        const char* const piece = mine + g * kFewLt + (m >> 2) * 32 + (m & 3) * 8;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < STEPS; ++u) {
            if (u > 0 && u % AB == 0) load_a(u);
            if (step_on(u)) {
                // A as it is (32 bytes a column, 16 columns a padded block), back through the transposing read: see fwd_prep_kernel
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const int kk = v * 32 + (lane >> 1);
                    *reinterpret_cast<u32x4*>(mine + (kk >> 4) * kFewLt + (kk & 15) * 32 + (lane & 1) * 16) = av[u % AB][v];
                }
                auto four = [&](int col0) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(piece + col0 * 32)); };
                const v4s e0 = four(0), e1 = four(4), o0 = four(8), o1 = four(12);
                const u32x4 even = __builtin_bit_cast(u32x4, (v8s){e0[0], e0[1], e0[2], e0[3], e1[0], e1[1], e1[2], e1[3]});
                const u32x4 odd = __builtin_bit_cast(u32x4, (v8s){o0[0], o0[1], o0[2], o0[3], o1[0], o1[1], o1[2], o1[3]});
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[u][0]), __builtin_bit_cast(bf16x8, even), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[u][1]), __builtin_bit_cast(bf16x8, odd), acc, 0, 0, 0);
            }
            if (u % SPS == SPS - 1) {
                if (has_slice(u / SPS)) *reinterpret_cast<f32x4*>(area + slice_id(u / SPS) * 1024 + lane * 16) = acc;
                acc = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    __syncthreads();

    // ---- row maxima; channel maxima of what; sums of the down-projection in slice order
    const lds_float* const csl = (const lds_float*)cs_copy;
    float mx = 0.0f;
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const int k = step_col(u) + g * 16;
        if (step_on(u) && k < c) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[8];
                widen_scale(xa[u][h], csl, k + h * 8, v);
#pragma unroll
                for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[e]));
            }
        }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lane < 16) rmax[wave][lane] = mx;
    if (n > 0) {
        float wmx = 0.0f;
#pragma unroll
        for (int i = 0; i < WV; ++i) {
            const int k = (tid + i * kFewThreads) / BN;
            if (k < n) {
                w_o[i] = __fmul_rn(sm1[k], w_o[i]);
                wmx = fmaxf(wmx, fabsf(w_o[i]));
            }
        }
        atomicMax(&wmaxbits[tid % BN], __float_as_uint(wmx));
    }
    if constexpr (HAS_LORA) {
        // element v of lane (p, q) is T[4 q + v][p]
        const int v = tid & 3, ln = (tid >> 2) & 63, p = tid >> 8;
        const int used = p ? na1 : na0;
        float sum = 0.0f;
        for (int w = 0; w < used; ++w) sum += *reinterpret_cast<const float*>(area + (p * kFewSlices + w) * 1024 + ln * 16 + v * 4);
        sum = sum * a.scale;
        const uint32_t hi = f32_to_bf16_rne(sum);
        tl[2 * p][(ln >> 4) * 4 + v][ln & 15] = (uint16_t)hi;
        tl[2 * p + 1][(ln >> 4) * 4 + v][ln & 15] = (uint16_t)f32_to_bf16_rne(sum - __uint_as_float(hi << 16));
    }
    __syncthreads();

    // ---- codes: of this wavefront's steps (kept in the registers), of the outlier columns, of what
    float cc;
    {
        float mrow = 0.0f, d;
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) mrow = fmaxf(mrow, rmax[w][m]);
        rtn_steps(mrow, d, cc);
        if (wave == 0 && lane < 16) {
            rowd[lane] = d;
            if (live && tn == 0) a.delta[row] = d;
        }
    }
    i32x4 xc[STEPS];
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const int k = step_col(u) + g * 16;
        xc[u] = (i32x4){0, 0, 0, 0};
        if (step_on(u) && k < c) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[8];
                widen_scale(xa[u][h], csl, k + h * 8, v);
                const u32x2 p = pack_codes(v, cc);
                xc[u][2 * h] = (int)p[0];
                xc[u][2 * h + 1] = (int)p[1];
            }
            // (the tiles of a row of tiles share the writing of its codes)
            if (live && (step_col(u) >> 6) % tiles_n == tn) *reinterpret_cast<i32x4*>(a.Xq + row * (int64_t)c + k) = xc[u];
        }
    }
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = wave * 8 + i * 4 + g;
            const int8_t q = (int8_t)(k < n ? rtn_code(__fmul_rn(bf16_bits_to_f32(xo[i]), rinv[k]), cc) : 0);
            xoc[m][k] = q;
        }
        static_assert(kFewThreads % BN == 0, "the elements of a thread are of one channel");
        const int jl = tid % BN;
        float d, cw;
        rtn_steps(__uint_as_float(wmaxbits[jl]), d, cw);
        if (tid < BN) dwh[jl] = d;
#pragma unroll
        for (int i = 0; i < WV; ++i) {
            const int k = (tid + i * kFewThreads) / BN;
            wcodes[jl][k] = (int8_t)(k < n ? rtn_code(w_o[i], cw) : 0);
        }
    }

    // ---- the product of this wavefront's steps
    i32x4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = (i32x4){0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        if (step_on(u)) {
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[u % PD][j], xc[u], acc[j], 0, 0, 0);
        }
        if (u + PD < STEPS) fetch_w(u + PD);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) *reinterpret_cast<i32x4*>(area + ((wave * NB + j) * 64 + lane) * 16) = acc[j];
    __syncthreads();

    // ---- epilogue: block b by wavefront b; the others write the rest
    if (wave < NB && wave * 16 < nlive) {
        i32x4 sum = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) sum += *reinterpret_cast<const i32x4*>(area + ((w * NB + wave) * 64 + lane) * 16);
        const int ch = wave * 16;
        i32x4 acc2 = {0, 0, 0, 0};
        float cs2[4] = {0.f, 0.f, 0.f, 0.f};
        if (n > 0) {
            acc2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const i32x4*>(&wcodes[ch + m][g * 16]),
                                                         *reinterpret_cast<const i32x4*>(&xoc[m][g * 16]), acc2, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) cs2[v] = dwh[ch + g * 4 + v];
        }
        f32x4 r = {0.f, 0.f, 0.f, 0.f};
        if constexpr (HAS_LORA) {
            const bf16x8 l = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(&bt[ch + m][(g & 1) * 8]));
#pragma unroll
            for (int part = 0; part < 2; ++part)
                r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    l, __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(&tl[2 * part + (g >> 1)][m][(g & 1) * 8])), r, 0, 0, 0);
        }
        const float rs = rowd[m];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float cs = dw[ch + g * 4 + v];
            r[v] = __builtin_fmaf(rs, __builtin_fmaf((float)sum[v], cs, (float)acc2[v] * cs2[v]), r[v]);
        }
        if (live) {
            float* const out = a.Y + row * a.ldy + n0 + ch + g * 4;
            if (a.ldy % 4 == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 15u) == 0) {
                *reinterpret_cast<f32x4*>(out) = r;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = r[v];
            }
        }
    }
    if (n == 0) return;
    if (blockIdx.y == 0) {
        for (int q = tid; q < nlive * 4; q += kFewThreads)
            *reinterpret_cast<i32x4*>(a.what_int + (int64_t)(n0 + (q >> 2)) * 64 + (q & 3) * 16) =
                *reinterpret_cast<const i32x4*>(&wcodes[q >> 2][(q & 3) * 16]);
        if (tid < nlive) a.delta_what[n0 + tid] = dwh[tid];
    }
    if (tn == 0 && tid >= 256 && tid < 256 + 64) {
        const int q = tid - 256, r = q >> 2;
        if (row0 + r < a.t)
            *reinterpret_cast<i32x4*>(a.xq_O + (row0 + r) * 64 + (q & 3) * 16) = *reinterpret_cast<const i32x4*>(&xoc[r][(q & 3) * 16]);
    }
    if (wave == kFewWaves - 1) {
        // this wavefront's mark has reached memory; are all there?
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bool all = true;
        for (int i = lane; i < groups; i += 64)
            all = all && __hip_atomic_load(&a.words[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
        if (__all(all)) {
            if (lane < n) {
                a.s_O[lane] = snew[lane];
                a.colscale[ocol] = rinv[lane];
                if (a.cmax_out) a.cmax_out[lane] = __uint_as_float(smax[lane]);
            }
            if (lane == 0) __hip_atomic_store(a.epoch, epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int i = lane; i < groups; i += 64)
                __hip_atomic_store(&a.words[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// The narrowest tiles that make a single round: up to 256 workgroups without outliers and 2048 columns (1024 without an adapter: 5 x 1456
// -> 336 6.6 / 7.3); with outliers, whose columns
// every workgroup gathers and whose words every workgroup reads, up to 64 workgroups, 1024 columns and 1024 gathered values.
// Of 292 forward steps of 1 to 512 rows and up to 2048 columns, every tile timed, the rule takes 151: 0.75 of the time of the two
// launches in the geometric mean, none more than 2 % slower; on 300 operand sets in turn 55 of them 0.69 (rank 16) and 0.72.  Beyond it, two launches / this one, us: 256 x 512 -> 512 with 8 outliers
// (128 workgroups) 12.1 / 12.4, 11 x 1792 -> 1024 with 5 11.6 / 11.4, 16 x 3072 -> 9216 with 31 outliers and rank 16 21.6 / 23.8
// (every workgroup quantizes 16 rows of 3072 columns, 3.5 us of vector instructions, and fetches them and A at 45 KB/us), 77 x 2944
// -> 576 without outliers 15.0 / 14.6.  With an adapter the product's order of summation must be this kernel's.
int fwd_few_blocks(int64_t t, int64_t c_in, int64_t c_out, int32_t n, int32_t r) {
    if ((r != 0 && r != 16) || n > 64 || c_in > (n > 0 || r == 0 ? 1024 : 2048) || (int64_t)n * t > 1024) return 0;
    for (int blocks = 1; blocks <= 4; blocks *= 2)
        if ((t + kFewRows - 1) / kFewRows * ((c_out + blocks * 16 - 1) / (blocks * 16)) <= (n > 0 ? 64 : 256))
            return r == 0 || gemm_takes_rows(t, c_out, c_in, r) ? blocks : 0;
    return 0;
}
int fwd_few_groups(int64_t t, int64_t c_out, int blocks) {
    return (int)((t + kFewRows - 1) / kFewRows * ((c_out + blocks * 16 - 1) / (blocks * 16)));
}

template <int SPS, int SL, int NB>
static hipError_t launch_few(bool lora, dim3 grid, hipStream_t stream, const FwdFewArgs& a, const int32_t* O) {
    auto k = lora ? fwd_few_kernel<SPS, SL, NB, true> : fwd_few_kernel<SPS, SL, NB, false>;
    const size_t red = lora ? 2 * kFewSlices * 1024 : 0, exchange = (size_t)kFewWaves * NB * 1024;
    const size_t lds = (((size_t)a.c * 4 + 255) & ~(size_t)255) + (lora ? (size_t)kFewWaves * 4 * kFewLt : 0) + (red > exchange ? red : exchange);
    if (lds > kPlainLds) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, grid, dim3(kFewThreads), lds, stream, a, O);
    return hipGetLastError();
}

template <int NB>
static hipError_t launch_few_steps(bool lora, dim3 grid, hipStream_t stream, const FwdFewArgs& a, const int32_t* O) {
    // slices as the kernel cuts them: steps of a slice, slices of a wavefront
    const int c = a.c, cp = (c + kLoraParts * 64 - 1) / (kLoraParts * 64) * 64, len0 = cp < c ? cp : c, len1 = c - len0;
    const int kw0 = (len0 + kFewSlices * 64 - 1) / (kFewSlices * 64) * 64, kw1 = (len1 + kFewSlices * 64 - 1) / (kFewSlices * 64) * 64;
    const int active = (len0 + kw0 - 1) / kw0 + (len1 > 0 ? (len1 + kw1 - 1) / kw1 : 0);
    const int sps = kw0 / 64, sl = (active + kFewWaves - 1) / kFewWaves;
    if (sps == 1 && sl == 1) return launch_few<1, 1, NB>(lora, grid, stream, a, O);
    if (sps == 1 && sl == 2) return launch_few<1, 2, NB>(lora, grid, stream, a, O);
    if (sps == 1) return launch_few<1, 4, NB>(lora, grid, stream, a, O);
    return hipErrorInvalidValue;
}

hipError_t launch_fwd_few(int blocks, const uint16_t* X, int64_t t, int64_t c, int64_t ldx, const int32_t* O, int32_t n,
                          const float* wmax_O, float gamma, float* s_O, float* colscale, float* cmax_out, const float* W_O,
                          int64_t c_out, int8_t* what_int, float* delta_what, int8_t* Xq, float* delta, int8_t* xq_O,
                          const int8_t* Wq, const float* delta_w, const uint16_t* A, const uint16_t* B, int32_t r, float scale,
                          float* Y, int64_t ldy, void* scratch, hipStream_t stream) {
    ProfScope prof(K_FWD_FEW, stream);
    FwdFewArgs a{};
    a.X = X; a.t = t; a.c = (int)c; a.ldx = ldx; a.n = n;
    a.wmax_O = wmax_O; a.gamma = gamma; a.s_O = s_O; a.colscale = colscale; a.cmax_out = cmax_out;
    a.W_O = W_O; a.c_out = (int)c_out; a.what_int = what_int; a.delta_what = delta_what;
    a.Xq = Xq; a.delta = delta; a.xq_O = xq_O;
    a.Wq = Wq; a.cpad = packed_weight_cpad(c); a.delta_w = delta_w;
    a.A = A; a.B = B; a.scale = scale; a.Y = Y; a.ldy = ldy;
    a.words = reinterpret_cast<uint64_t*>(static_cast<char*>(scratch) + kFwdPrepWordsAt);
    a.epoch = reinterpret_cast<uint64_t*>(scratch);
    const dim3 grid((unsigned)((c_out + blocks * 16 - 1) / (blocks * 16)), (unsigned)((t + kFewRows - 1) / kFewRows));
    if (blocks == 1) return launch_few_steps<1>(r == 16, grid, stream, a, O);
    if (blocks == 2) return launch_few_steps<2>(r == 16, grid, stream, a, O);
    return launch_few_steps<4>(r == 16, grid, stream, a, O);
}

}  // namespace quaff
