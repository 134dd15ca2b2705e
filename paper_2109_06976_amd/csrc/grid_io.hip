// Copy kernel of the host calls (grid_fd_grad_mapped; small batches of grid_fd_grad_pinned and
// grid_fd_grad_host, both ways): moves packed arrays between device memory and pinned host
// memory through its device mapping, so that the transfer is
// a kernel's stores over the host link rather than a copy-engine job (whose start-up latency
// dominates transfers of the few hundred kilobytes a batch of knots produces).
//
// Each thread moves 16 bytes per step (dwordx4 load and store) over a grid-stride loop; the
// tail of n mod 4 floats is moved one float per thread by the first threads.
//
// With `stamps` each workgroup leaves the device clock at its start and once its stores have
// arrived (they go through the caches: otherwise they wait there for the kernel's end, and 158 KB
// seem to cross the link in 0.9 us). The phases of a host call are timed so, where an event
// between two kernels holds the stream up for about 3 us: chain7 at 16, 256 and 1024 knots by
// grid_fd_grad_host 32.2 / 37.3 / 57.8 us with events, 22.8 / 29.3 / 53.8 here; a fence of the
// system's scope in place of such stores 23.5 / 32.1 / 66.4.
#include <hip/hip_runtime.h>

#include "grid_internal.h"

typedef unsigned Words __attribute__((ext_vector_type(4)));
constexpr int kThrough = 1 | 16;   // sc0 | sc1: a store of the system's scope

extern "C" __global__ void __launch_bounds__(256)
grid_copy_out_kernel(const float4* __restrict__ src, float4* __restrict__ dst, long n4,
                     const float* __restrict__ src_tail, float* __restrict__ dst_tail, int tail,
                     ulonglong2* __restrict__ stamps)
{
    const unsigned long long begin = stamps ? wall_clock64() : 0;
    const long stride = (long)gridDim.x * blockDim.x;
    const long first = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (stamps) {                                      // (n4 < 2^27)
        const auto out = __builtin_amdgcn_make_buffer_rsrc(dst, 0, (int)(n4 * 16), 0x00027000);
        for (long i = first; i < n4; i += stride) {
            const float4 v = src[i];
            __builtin_amdgcn_raw_buffer_store_b128(
                Words{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z),
                      __float_as_uint(v.w)},
                out, (int)(i * 16), 0, kThrough);
        }
    } else {
        for (long i = first; i < n4; i += stride)
            dst[i] = src[i];
    }
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t < tail)
        dst_tail[t] = src_tail[t];
    if (stamps) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0)
            stamps[blockIdx.x] = ulonglong2{begin, (unsigned long long)wall_clock64()};
    }
}

namespace grid_impl {

int copy_blocks(size_t n)
{
    const size_t blocks = (n / 4 + 255) / 256;
    return blocks < 1 ? 1 : (blocks > kMaxCopyBlocks ? kMaxCopyBlocks : (int)blocks);
}

hipError_t launch_copy_out(const float* src, float* dst, size_t n, hipStream_t stream,
                           uint64_t* stamps)
{
    // both buffers start 16-byte aligned (device allocation, pinned host allocation)
    const long n4 = (long)(n / 4);
    const int tail = (int)(n % 4);
    const int blocks = copy_blocks(n);
    hipLaunchKernelGGL(grid_copy_out_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                       reinterpret_cast<const float4*>(src), reinterpret_cast<float4*>(dst), n4,
                       src + 4 * n4, dst + 4 * n4, tail, reinterpret_cast<ulonglong2*>(stamps));
    return hipGetLastError();
}

}  // namespace grid_impl
