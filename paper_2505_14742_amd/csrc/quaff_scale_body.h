// Device code of the outlier-column abs-max (Eq. 8 of the paper, max_i |X[i, O_k]|), shared by its stand-alone launch
// and by the launch that runs it next to the LoRA down-projection.
#pragma once
#include "quaff_internal.h"

namespace quaff {

constexpr int kRowsPerSlab = 16;
constexpr int kMaxSlabs = 128;

// part[slab][k] = max over the slab's rows of |X[row, O_k]|; slab s owns the 16-row groups s, s + nslab, ...
// Work of workgroup `block` of `nslab` (all NT threads take part).  Sixteen outlier columns are handled per pass:
// thread (slot = tid / 16, kk = tid % 16) walks rows slot, slot + NT / 16, ... of the slab's groups for column kk of the
// pass - sixteen neighbouring lanes read sixteen (often neighbouring) columns of one row - and keeps a running maximum
// in a register, four gathers in flight.  The maxima of a wavefront's four row slots are combined with wavefront
// shuffles and the wavefronts' results through a small LDS array (plain stores, one barrier): no atomics.
// wred is 16 * NT / 64 words of LDS.
template <int NT>
__device__ __forceinline__ void colmax_outlier_body(int block, int nslab, uint32_t* wred, const uint16_t* __restrict__ X,
                                                    int64_t t, int64_t ldx, const int32_t* __restrict__ O, int n,
                                                    uint32_t* __restrict__ part, const float* __restrict__ s_O,
                                                    float* __restrict__ s_prev) {
    constexpr int SLOTS = NT / 16, NWAVE = NT / 64;
    static_assert(SLOTS % kRowsPerSlab == 0, "the row slots of a pass cover whole 16-row groups");
    if (block == 0)
        for (int k = threadIdx.x; k < n; k += NT) s_prev[k] = s_O[k];
    const int kk = threadIdx.x & 15, slot = threadIdx.x >> 4;
    // row of this thread in its first pass over the slab's groups, and the distance between passes: the slab's
    // groups are 16 rows every nslab * 16 rows; the SLOTS row slots of a pass cover SLOTS / 16 of them
    constexpr int GPP = SLOTS / kRowsPerSlab;     // groups per pass
    const int64_t group_stride = (int64_t)nslab * kRowsPerSlab;
    for (int k0 = 0; k0 < n; k0 += 16) {
        const int k = k0 + kk < n ? k0 + kk : n - 1;
        const int64_t col = O[k];
        uint32_t mx = 0;
        const int64_t first = ((int64_t)block + (int64_t)(slot / kRowsPerSlab) * nslab) * kRowsPerSlab + slot % kRowsPerSlab;
        const int64_t step = group_stride * GPP;
        for (int64_t row = first; row < t; row += 4 * step) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t r = row + u * step;
                v[u] = (uint32_t)X[(r < t ? r : t - 1) * ldx + col] & 0x7FFFu;   // (a repeated row changes no maximum)
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) mx = v[u] > mx ? v[u] : mx;
        }
        // the four row slots of a wavefront, then the wavefronts
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 16, 64));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 32, 64));
        if ((threadIdx.x & 63) < 16) wred[(threadIdx.x >> 6) * 16 + kk] = mx;
        __syncthreads();
        if (threadIdx.x < 16 && k0 + kk < n) {
            uint32_t m = 0;
#pragma unroll
            for (int w = 0; w < NWAVE; ++w) m = max(m, wred[w * 16 + kk]);
            part[(int64_t)block * n + k0 + kk] = m << 16;                              // |x| as fp32 bits
        }
        __syncthreads();
    }
}

// Dense variant of the column abs-max for outlier sets that touch most 64-byte segments of a row anyway (the
// paper's 4 % - 10 % budgets): every column of a 2048-column chunk is reduced over the slab's rows with coalesced
// 16-byte loads (bf16 magnitudes compare as integers), then the chunk's outlier columns are picked out of LDS.
// Four groups of 256 threads share a slab's rows: as many loads in flight as with four times the slabs, whose partial
// maxima every workgroup of the next launch would have to fold.
constexpr int kDenseGroups = 4, kDenseThreads = 256 * kDenseGroups;
__device__ __forceinline__ void colmax_dense_body(int chunk, int slab, uint16_t (*cm)[2048] /* LDS [kDenseGroups] */,
                                                  const uint16_t* __restrict__ X, int64_t t, int64_t c_in, int64_t ldx,
                                                  const int32_t* __restrict__ O, int n, uint32_t* __restrict__ part,
                                                  const float* __restrict__ s_O, float* __restrict__ s_prev, int rows_per_slab) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __shared__ int krange[2];
    const int chunk0 = chunk * 2048;
    const int lane = threadIdx.x & 255, grp = threadIdx.x >> 8;
    if (chunk == 0 && slab == 0)
        for (int k = threadIdx.x; k < n; k += kDenseThreads) s_prev[k] = s_O[k];
    if (threadIdx.x < 2) {
        // first outlier index >= chunk0 (thread 0) and >= chunk0 + 2048 (thread 1): O is sorted
        const int target = chunk0 + 2048 * (int)threadIdx.x;
        int lo = 0, hi = n;
        while (lo < hi) {
            int mid = (lo + hi) >> 1;
            if (O[mid] < target) lo = mid + 1; else hi = mid;
        }
        krange[threadIdx.x] = lo;
    }
    const int64_t col = chunk0 + (int64_t)lane * 8;
    const int64_t r0 = (int64_t)slab * rows_per_slab;
    const int64_t r1 = r0 + rows_per_slab < t ? r0 + rows_per_slab : t;
    uint32_t mx[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (col < c_in) {
        const uint16_t* src = X + col;
        for (int64_t row = r0 + grp; row < r1; row += 4 * kDenseGroups) {   // four independent loads in flight
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t rr = row + u * kDenseGroups < r1 ? row + u * kDenseGroups : r1 - 1;
                v[u] = *reinterpret_cast<const u32x4*>(src + rr * ldx);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {     // a repeated row changes no maximum
                    uint32_t lo = v[u][w] & 0x7FFFu, hi = (v[u][w] >> 16) & 0x7FFFu;
                    mx[2 * w] = lo > mx[2 * w] ? lo : mx[2 * w];
                    mx[2 * w + 1] = hi > mx[2 * w + 1] ? hi : mx[2 * w + 1];
                }
        }
    }
    u32x4 packed;
#pragma unroll
    for (int w = 0; w < 4; ++w) packed[w] = mx[2 * w] | (mx[2 * w + 1] << 16);
    *reinterpret_cast<u32x4*>(&cm[grp][lane * 8]) = packed;
    __syncthreads();
    for (int k = krange[0] + threadIdx.x; k < krange[1]; k += kDenseThreads) {
        const int at = O[k] - chunk0;
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < kDenseGroups; ++u) m = max(m, (uint32_t)cm[u][at]);
        part[(int64_t)slab * n + k] = m << 16;                              // |x| as fp32 bits
    }
}

// Eq. 7 with Eq. 8 for one outlier channel, in fp32 with one rounding per operation
__device__ __forceinline__ float momentum_scale(float cmax, float wmax, float s_prev, float gamma) {
    float beta = 1.0f;
    if (wmax > 0.0f) beta = fmaxf(1.0f, __builtin_sqrtf(__fdiv_rn(cmax, wmax)));                 // Eq. 8
    return __fadd_rn(__fmul_rn(gamma, s_prev), __fmul_rn(__fsub_rn(1.0f, gamma), beta));       // Eq. 7
}

// Work of workgroup `block` (NT threads): reduce the partial maxima, evaluate Eq. 8 / Eq. 7 for all outlier channels (workgroup 0
// publishes s, 1/s and cmax), requantize what.  A workgroup owns 16 output channels; its NT / 16 thread
// groups take four consecutive outliers of every NT / 4, NB times.  What bounds it is the chain of memory round trips, so both long
// reads are in flight at once: this workgroup's part of W_O (kept in registers, one sweep instead of one for the maxima
// and one for the codes) and the partial maxima, folded with one column of them per thread (coalesced, an LDS atomic per
// thread instead of one per partial maximum).  The codes leave through LDS: sixteen output channels are contiguous in what_int.
// HELD = false: more outliers than NB NT / 4, which a second sweep of W_O fetches again.
// Measured at 2048 x 8192 -> 3072 with 819 outliers: 11.2 us, at 2048 x 3072 -> 3072 with 31 (256 threads) 4.0 and at 13824 channels
// with 64 outliers 6.5; with a thread per channel, which walks the outliers in a chain, 8.2 and 13.4.  At 819 outliers with 32 channels a workgroup, 128 slabs of partial maxima
// folded with one LDS atomic each and W_O swept twice in chains of eight loads 34.7 us.
constexpr int kWideCh = 16;
template <int NT, int NB, bool HELD>
__device__ __forceinline__ void momentum_what_body(int block, uint32_t* smax /* LDS [n]: maxima, then s_k - 1 */,
                                                   const uint32_t* __restrict__ part, int nslab, int n, int n_pad,
                                                   const float* __restrict__ wmax_O, const float* __restrict__ s_prev, float gamma,
                                                   const int32_t* __restrict__ O, float* __restrict__ s_O,
                                                   float* __restrict__ colscale, float* __restrict__ cmax_out,
                                                   const float* __restrict__ W_O, int64_t c_out, int8_t* __restrict__ what_int,
                                                   float* __restrict__ delta_what) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int GROUPS = NT / kWideCh, SPAN = 4 * GROUPS * NB;        // outliers per sweep
    constexpr int ROW = SPAN + 16;                                  // LDS row of codes: 16 channels in 16 different banks
    __shared__ __attribute__((aligned(16))) uint32_t codes[kWideCh * ROW / 4];
    __shared__ float red[NT / 64][kWideCh];
    float* const sm1 = reinterpret_cast<float*>(smax);
    const int jj = threadIdx.x % kWideCh, grp = threadIdx.x / kWideCh;
    const int64_t j0 = (int64_t)block * kWideCh, j = j0 + jj;
    const int64_t jc = j < c_out ? j : c_out - 1;
    float w[NB][4];
    auto first_k = [&](int base, int b) { return base + (b * GROUPS + grp) * 4; };
    auto load = [&](int base) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = first_k(base, b) + u;
                w[b][u] = W_O[(int64_t)(k < n ? k : n - 1) * c_out + jc];
            }
    };
    if (HELD) load(0);
    for (int k = threadIdx.x; k < n; k += NT) smax[k] = 0u;
    __syncthreads();
    // thread (share, k): column k of the slabs share, share + shares, ...
    const int width = n < NT ? (n + 63) / 64 * 64 : NT, shares = NT / width;
    const int share = threadIdx.x / width;
    for (int k = threadIdx.x % width; k < n && share < shares; k += width) {
        uint32_t m = 0u;
        for (int s0 = share; s0 < nslab; s0 += 16 * shares) {
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int sl = s0 + u * shares;                     // (a repeated slab changes no maximum)
                v[u] = part[(int64_t)(sl < nslab ? sl : s0) * n + k];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) m = max(m, v[u]);
        }
        atomicMax(&smax[k], m);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += NT) {
        const float cmax = __uint_as_float(smax[k]);
        const float s = momentum_scale(cmax, wmax_O[k], s_prev[k], gamma);
        sm1[k] = __fsub_rn(s, 1.0f);
        if (block == 0) {
            s_O[k] = s;
            colscale[O[k]] = __fdiv_rn(1.0f, s);
            if (cmax_out) cmax_out[k] = cmax;
        }
    }
    __syncthreads();
    // max_k |what[k, j]|: this thread's share, the wavefront's four groups, the wavefronts
    float m = 0.0f;
    for (int base = 0; base < n; base += SPAN) {
        if (!HELD) load(base);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = first_k(base, b) + u;
                const float v = k < n ? __fmul_rn(sm1[k < n ? k : 0], w[b][u]) : 0.0f;
                if (HELD) w[b][u] = v;
                m = fmaxf(m, fabsf(v));
            }
        if (HELD) break;
    }
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if ((threadIdx.x & 63) < kWideCh) red[threadIdx.x >> 6][jj] = m;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NT / 64; ++v) m = fmaxf(m, red[v][jj]);
    float d, c;
    rtn_steps(m, d, c);
    if (grp == 0 && j < c_out) delta_what[j] = d;
    const int channels = c_out - j0 < kWideCh ? (int)(c_out - j0) : kWideCh;
    for (int base = 0; base < n_pad; base += SPAN) {
        if (!HELD) load(base);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int k0 = first_k(base, b);
            uint32_t q = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + u;
                float v = w[b][u];
                if (!HELD) v = k < n ? __fmul_rn(sm1[k < n ? k : 0], v) : 0.0f;
                q |= (uint32_t)(rtn_code(v, c) & 0xFF) << (8 * u);  // (zero beyond n: code 0)
            }
            codes[(jj * ROW + k0 - base) >> 2] = q;
        }
        __syncthreads();
        const int span = n_pad - base < SPAN ? n_pad - base : SPAN, per_row = span / 16;   // 16-byte chunks
        for (int e = threadIdx.x; e < channels * per_row; e += NT) {
            const int row = e / per_row, at = (e - row * per_row) * 16;
            *reinterpret_cast<u32x4*>(what_int + (j0 + row) * n_pad + base + at) =
                *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(codes) + row * ROW + at);
        }
        if (HELD) break;
        __syncthreads();
    }
}

}  // namespace quaff
