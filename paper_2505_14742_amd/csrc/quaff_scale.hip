// Targeted momentum scaling (Eq. 7, Eq. 8 of the paper) and the dynamic outlier weights
// what = (s_O - 1) W_O with their per-output-channel quantization (Eq. 5, Eq. 9).
//
// Two launches:
//   colmax_outlier_kernel   partial column maxima of |X[:, O]| per slab of rows (a strided 2-byte gather: the
//                           traffic is one DRAM sector per (row, outlier) whatever the kernel does; register maxima
//                           combined with wavefront shuffles), and a copy
//                           of the previous scales so that the in-place update below has no read/write race;
//   momentum_what_kernel    every block reduces the partial maxima and evaluates Eq. 8 / Eq. 7 for all outlier
//                           channels (a few hundred flops, cheaper than another launch); block 0 publishes s,
//                           1/s and cmax; then the block requantizes sixteen output channels of what.
// Maxima of non-negative floats are taken on their bit patterns (same order as unsigned integers), which is exact
// and independent of the order in which they are combined.
#include "quaff_scale_body.h"
#include <mutex>

namespace quaff {

// Scratch of quaff_scale_update_static (callers that cannot allocate): the partial column maxima [slabs x n] and the
// copy of the previous scales [n] that the workspace of quaff_scale_update otherwise holds.  One copy per device, held
// until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; kernels get the
// address that call returns.
constexpr int kStaticMaxOutliers = 1024;
static __device__ __align__(256) __attribute__((used)) float scratch[(size_t)(kMaxSlabs + 1) * kStaticMaxOutliers];

int scale_update_static_max_outliers() { return kStaticMaxOutliers; }

hipError_t scale_update_static_scratch(float** ptr) {
    static std::mutex mu;
    static float* per_device[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // this device's copy of the array
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        per_device[dev] = static_cast<float*>(p);
    }
    *ptr = per_device[dev];
    return hipSuccess;
}

constexpr int kPartWords = 4096;    // partial maxima that a workgroup of momentum_what_kernel folds

int scale_update_blocks(int64_t t) {
    int64_t b = (t + kRowsPerSlab - 1) / kRowsPerSlab;
    return (int)(b < kMaxSlabs ? b : kMaxSlabs);
}

__global__ void __launch_bounds__(256)
colmax_outlier_kernel(const uint16_t* __restrict__ X, int64_t t, int64_t ldx, const int32_t* __restrict__ O, int n,
                      uint32_t* __restrict__ part, const float* __restrict__ s_O, float* __restrict__ s_prev) {
    __shared__ uint32_t wred[16 * 256 / 64];
    colmax_outlier_body<256>(blockIdx.x, gridDim.x, wred, X, t, ldx, O, n, part, s_O, s_prev);
}

__global__ void __launch_bounds__(kDenseThreads)
colmax_dense_kernel(const uint16_t* __restrict__ X, int64_t t, int64_t c_in, int64_t ldx, const int32_t* __restrict__ O,
                    int n, uint32_t* __restrict__ part, const float* __restrict__ s_O, float* __restrict__ s_prev,
                    int rows_per_slab) {
    __shared__ __attribute__((aligned(16))) uint16_t cm[kDenseGroups][2048];
    colmax_dense_body(blockIdx.x, blockIdx.y, cm, X, t, c_in, ldx, O, n, part, s_O, s_prev, rows_per_slab);
}

template <int NT, int NB, bool HELD>
__global__ void __launch_bounds__(NT)
momentum_what_kernel(const uint32_t* __restrict__ part, int nslab, int n, int n_pad,
                     const float* __restrict__ wmax_O, const float* __restrict__ s_prev, float gamma,
                     const int32_t* __restrict__ O, float* __restrict__ s_O, float* __restrict__ colscale,
                     float* __restrict__ cmax_out, const float* __restrict__ W_O, int64_t c_out,
                     int8_t* __restrict__ what_int, float* __restrict__ delta_what) {
    extern __shared__ uint32_t smax[];                              // [n]
    momentum_what_body<NT, NB, HELD>(blockIdx.x, smax, part, nslab, n, n_pad, wmax_O, s_prev, gamma, O, s_O, colscale, cmax_out, W_O,
                                     c_out, what_int, delta_what);
}

// Validity of an outlier index list (Sec. 3.3 fixes O before fine-tuning: one check per layer).  One workgroup scans
// the list; *result = 0 when O is strictly ascending and inside [0, c_in), else 1 + the first offending position.
__global__ void __launch_bounds__(256)
check_outliers_kernel(const int32_t* __restrict__ O, int n, int64_t c_in, int32_t* __restrict__ result) {
    __shared__ int first_bad;
    if (threadIdx.x == 0) first_bad = 0x7FFFFFFF;
    __syncthreads();
    int mine = 0x7FFFFFFF;
    for (int k = threadIdx.x; k < n; k += 256) {
        const int64_t v = O[k];
        const bool bad = v < 0 || v >= c_in || (k > 0 && (int64_t)O[k - 1] >= v);
        if (bad && k < mine) mine = k;
    }
    if (mine != 0x7FFFFFFF) atomicMin(&first_bad, mine);
    __syncthreads();
    if (threadIdx.x == 0) *result = first_bad == 0x7FFFFFFF ? 0 : first_bad + 1;
}

hipError_t launch_check_outliers(const int32_t* O, int32_t n, int64_t c_in, int32_t* result, hipStream_t stream) {
    hipLaunchKernelGGL(check_outliers_kernel, dim3(1), dim3(256), 0, stream, O, n, c_in, result);
    return hipGetLastError();
}

// as many slabs as the rows allow, but no more partial maxima than that
int scale_update_gather_slabs(int64_t t, int32_t n) {
    int nslab = scale_update_blocks(t);
    const int cap = kPartWords / n > 16 ? kPartWords / n : 16;
    return nslab < cap ? nslab : cap;
}

// one (chunk, slab) workgroup per compute unit, within the slab count the workspace was sized for
int scale_update_dense_slabs(int64_t t, int64_t c_in, int* chunks, int* rows) {
    *chunks = (int)((c_in + 2047) / 2048);
    const int want = (256 + *chunks - 1) / *chunks, most = scale_update_blocks(t), nslab = want < most ? want : most;
    *rows = (int)((t + nslab - 1) / nslab);
    return (int)((t + *rows - 1) / *rows);
}

hipError_t launch_scale_update(const uint16_t* X, int64_t t, int64_t c_in, int64_t ldx, const int32_t* O, int32_t n,
                               const float* W_O, const float* wmax_O, int64_t c_out, float gamma, float* s_O,
                               float* colscale, int8_t* what_int, float* delta_what, float* cmax_out, float* ws,
                               hipStream_t stream) {
    const int n_pad = (n + kPadK - 1) / kPadK * kPadK;
    uint32_t* part = reinterpret_cast<uint32_t*>(ws);   // [nslab x n]
    int nslab = scale_update_blocks(t);
    const bool dense = (int64_t)n * 64 >= c_in;          // most 64-byte segments of a row hold an outlier anyway
    if (dense) {
        int chunks, rows;
        nslab = scale_update_dense_slabs(t, c_in, &chunks, &rows);
        float* s_prev = ws + (int64_t)nslab * n;
        {
            ProfScope prof(K_COLMAX, stream);
            hipLaunchKernelGGL(colmax_dense_kernel, dim3(chunks, nslab), dim3(kDenseThreads), 0, stream, X, t, c_in, ldx, O, n,
                               part, s_O, s_prev, rows);
        }
        return launch_momentum(part, nslab, n, n_pad, wmax_O, s_prev, gamma, O, s_O, colscale, cmax_out, W_O, c_out,
                               what_int, delta_what, stream);
    }
    nslab = scale_update_gather_slabs(t, n);
    float* s_prev = ws + (int64_t)nslab * n;            // [n]
    {
        ProfScope prof(K_COLMAX, stream);
        hipLaunchKernelGGL(colmax_outlier_kernel, dim3(nslab), dim3(256), 0, stream, X, t, ldx, O,
                           n, part, s_O, s_prev);
    }
    return launch_momentum(part, nslab, n, n_pad, wmax_O, s_prev, gamma, O, s_O, colscale, cmax_out, W_O, c_out,
                           what_int, delta_what, stream);
}

hipError_t launch_momentum(const uint32_t* part, int nslab, int n, int n_pad, const float* wmax_O,
                                  const float* s_prev, float gamma, const int32_t* O, float* s_O, float* colscale,
                                  float* cmax_out, const float* W_O, int64_t c_out, int8_t* what_int,
                                  float* delta_what, hipStream_t stream) {
    ProfScope prof(K_MOMENTUM, stream);
    {
        const size_t lds = (size_t)n * sizeof(uint32_t);
        const dim3 grid((unsigned)((c_out + kWideCh - 1) / kWideCh));
#define QUAFF_WIDE(NT, NB, HELD)                                                                                      \
    {                                                                                                                 \
        auto k = momentum_what_kernel<NT, NB, HELD>;                                                             \
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),                                          \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                     \
        if (e != hipSuccess) return e;                                                                                \
        hipLaunchKernelGGL(k, grid, dim3(NT), lds, stream, part, nslab, n, n_pad, wmax_O, s_prev, gamma, O, s_O,      \
                           colscale, cmax_out, W_O, c_out, what_int, delta_what);                                     \
    }
        // The smallest number of registers that holds a thread's share of W_O; beyond 2048 outliers it is fetched twice.  Up to
        // 256 outliers half the threads hold as much with one register set more, and more workgroups fit a compute unit:
        // scale updates of 46 tokens, us, 1024 / 512 threads: 65 outliers, 3072 channels 7.4 / 7.2, 13648 channels 11.9 / 8.9; 158
        // outliers 7.8 / 7.6 and 13.0 / 10.2.  With more maxima to fold and every workgroup resident 1024 are faster: 2048 tokens,
        // 256 outliers, 4096 channels 9.5 / 9.8, 11008 channels 15.0 / 13.7.
        const bool resident = c_out <= 256 * kWideCh;
        if (n <= 64) QUAFF_WIDE(256, 1, true)
        else if (n <= 128) QUAFF_WIDE(512, 1, true)
        else if (n <= 256 && !resident) QUAFF_WIDE(512, 2, true)
        else if (n <= 256) QUAFF_WIDE(1024, 1, true)
        else if (n <= 512) QUAFF_WIDE(1024, 2, true)
        else if (n <= 1024) QUAFF_WIDE(1024, 4, true)
        else if (n <= 2048) QUAFF_WIDE(1024, 8, true)
        else QUAFF_WIDE(1024, 8, false)
#undef QUAFF_WIDE
    }
    return hipGetLastError();
}

}  // namespace quaff
