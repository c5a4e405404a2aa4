// Generic exact-arithmetic path: fp32 FMA only (no matrix cores, no reduced precision), any n,
// any d <= 512, any block edge for the block mask.  It serves what the matrix-core kernels of the same arithmetic do not
// take.  One wavefront owns one row (attn_rows.hpp).
// Formulas: A, l, f, O, q, p of App. B.4 with the scale, mask and log-sum-exp readings.
#include "attn_rows.hpp"

namespace attn {

constexpr int kMaxD = 512;

// Four rows per workgroup, one per wave; false past the last row.
__device__ __forceinline__ bool wave_row(const GenericParams& p, int& bh, int& i) {
    const long r = (long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bh = (int)(r / p.n);
    i = (int)(r % p.n);
    return r < (long)p.batch * p.heads * p.n;
}

template <typename T, int D>  // d <= D
__global__ void __launch_bounds__(kThreads) generic_fwd_kernel(GenericParams p) {
    __shared__ float qs[4][D];
    int bh, i;
    if (wave_row(p, bh, i)) row_forward<T, row_words<T>(D)>(p, bh, i, threadIdx.x & 63, qs[threadIdx.x >> 6]);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) generic_delta_kernel(GenericParams p) {
    int bh, i;
    if (!wave_row(p, bh, i)) return;
    const float s = row_delta<T>(p, bh, i, threadIdx.x & 63);
    if ((threadIdx.x & 63) == 0) p.delta[(long)bh * p.n + i] = s;
}

template <typename T, int D>  // d <= D
__global__ void __launch_bounds__(kThreads) generic_dq_kernel(GenericParams p) {
    __shared__ float qs[4][D], gs[4][D];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bh, i;
    if (wave_row(p, bh, i)) row_dq<T, row_words<T>(D)>(p, bh, i, threadIdx.x & 63, p.delta[(long)bh * p.n + i], qs[w], gs[w]);
}

template <typename T, int D>  // d <= D
__global__ void __launch_bounds__(kThreads) generic_dkdv_kernel(GenericParams p) {
    __shared__ float ks[4][D], vs[4][D];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bh, j;
    if (!wave_row(p, bh, j)) return;
    row_dkdv<T, row_words<T>(D), false>(p, bh, j, threadIdx.x & 63, ks[w], vs[w]);
}

// delta[b, h, i] (p.O_in, p.dO, p.delta), any d
static void launch_generic_delta(bool is_bf16, const GenericParams& p, hipStream_t stream) {
    const dim3 grid((unsigned)(((long)p.batch * p.heads * p.n + 3) / 4));
    if (is_bf16) hipLaunchKernelGGL(generic_delta_kernel<__bf16>, grid, dim3(kThreads), 0, stream, p);
    else hipLaunchKernelGGL(generic_delta_kernel<float>, grid, dim3(kThreads), 0, stream, p);
}

template <typename T, int D>
static hipError_t run_generic(const GenericParams& p, bool backward, hipStream_t stream) {
    const long rows = (long)p.batch * p.heads * p.n;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(kThreads);
    if (!backward) {
        hipLaunchKernelGGL((generic_fwd_kernel<T, D>), grid, block, 0, stream, p);
    } else {
        launch_generic_delta(sizeof(T) == 2, p, stream);
        hipLaunchKernelGGL((generic_dq_kernel<T, D>), grid, block, 0, stream, p);
        hipLaunchKernelGGL((generic_dkdv_kernel<T, D>), grid, block, 0, stream, p);
    }
    return hipGetLastError();
}

template <typename T>
static hipError_t run_width(const GenericParams& p, bool backward, hipStream_t stream) {
    if (p.d <= 128) return run_generic<T, 128>(p, backward, stream);
    if (p.d <= 256) return run_generic<T, 256>(p, backward, stream);
    return run_generic<T, kMaxD>(p, backward, stream);
}

hipError_t launch_generic(bool is_bf16, bool backward, const GenericParams& p, hipStream_t stream) {
    if (p.d > kMaxD) return hipErrorInvalidValue;
    if (stream_takes(is_bf16, backward, p)) return launch_stream(is_bf16, backward, p, stream);
    return is_bf16 ? run_width<__bf16>(p, backward, stream) : run_width<float>(p, backward, stream);
}

}  // namespace attn
