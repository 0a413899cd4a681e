// Expert weights from pinned host memory into a staging slot (Sec. 4.2: prefetch of the next experts' weights).
//
// Bound by the host link.  A copy engine takes one matrix at a time and leaves the link idle between two of them, which for
// matrices of a few MB is a tenth of the time; a kernel reads all matrices of a group in one launch.  1.1 GB in matrices of
// 5.8 MB: 21.2 ms by copy engine (52.3 GB/s), 19.4 ms here (57.0 GB/s = one engine copy of 138 MB, the link's rate).  Few
// workgroups fill the link (8: 55.8 GB/s, 16: 57.0, 64: 57.3), and each takes a CU from the GEMM tiles of the group before.
#include "common.h"

namespace moe {
namespace {

constexpr int COPY_BLOCKS = 16;
constexpr int COPY_AHEAD = 4;       // 16-byte loads a thread has in flight
constexpr int COPY_PIECE = 4096;    // bytes that a workgroup's 256 threads load at once; a matrix is a multiple of it

// 16 bytes of host memory at base + off, past all caches: the host may have written them since an earlier launch read them, and
// not every kind of pinned memory is kept coherent with them.
__device__ __forceinline__ u32x4 load_host(const void* base, const uint32_t bytes, const uint32_t off) {
    u32x4 v = {0u, 0u, 0u, 0u};
#if defined(__gfx950__)
    constexpr int SYSTEM = 1 | 2 | 16;   // sc0 nt sc1
    v = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000), off, 0, SYSTEM);
#endif
    return v;
}

__global__ __launch_bounds__(256) void host_copy_kernel(const HostMatrices m) {
    const uint32_t per = m.bytes / COPY_PIECE, total = per * (uint32_t)m.n;
    const uint32_t at = threadIdx.x * 16;
    for (uint32_t p0 = blockIdx.x * COPY_AHEAD; p0 < total; p0 += COPY_BLOCKS * COPY_AHEAD) {
        u32x4 v[COPY_AHEAD];
#pragma unroll
        for (int u = 0; u < COPY_AHEAD; ++u) {
            const uint32_t p = min(p0 + u, total - 1), i = p / per;
            v[u] = load_host(m.src[i], m.bytes, (p - i * per) * COPY_PIECE + at);
        }
#pragma unroll
        for (int u = 0; u < COPY_AHEAD; ++u)
            if (p0 + u < total) *(u32x4*)(m.dst + (size_t)(p0 + u) * COPY_PIECE + at) = v[u];
    }
}

}  // namespace

hipError_t launch_host_copy(const HostMatrices& m, hipStream_t st) {
    if (m.n < 1 || m.n > HOST_MATRICES || m.bytes % COPY_PIECE || (uint64_t)m.bytes * m.n / COPY_PIECE >= (1u << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(host_copy_kernel, dim3(COPY_BLOCKS), dim3(256), 0, st, m);
    return hipGetLastError();
}

}  // namespace moe
