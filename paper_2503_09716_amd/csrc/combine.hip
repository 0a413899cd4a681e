// Weighted combine back to token order, and the one-time weight packing.
// (Sec. 2: the layer output is the weighted sum of the k experts' outputs, plus the shared
// expert every token passes through.)
//
// combine: one thread per token and 4 or 8 consecutive hidden elements (combine_elements), which gathers the k expert
// rows of its token through inv_perm, all of them in flight at once.  Sums are fp32 in the fixed order j = 0..k-1 then
// shared, every output element is written exactly once: no atomics, and the result is bit-identical from run to run.
// HBM-bound: reads k+1 rows, writes 1 row per token.  (moe_layer has this launch unless its shared experts' down GEMM does the work,
// launch_down_combine; the two larger layers below then make it in staged, streamed and fp32-y_perm calls only.)  Against one workgroup per token that walked its row 8 elements per
// thread and waited for each expert's row before it asked for the next: 160 experts top-6 + 2 shared, H = 5120, 32768
// tokens 614 -> 500 to 545 us by box (3.0 GB = 5.5 to 6.0 TB/s), 64 experts, H = 2048, 16384 tokens 120 -> 94 us, 1 token
// 2 us less of the layer's 47.
#include "common.h"

namespace moe {
namespace {

// N consecutive elements of a row, starting at element N*c, as they are stored.  NT: non-temporal
template <bool F32, int N, bool NT>
struct Piece {
    typedef uint32_t words __attribute__((ext_vector_type(N * (F32 ? 4 : 2) / 4)));
    words v;
    __device__ __forceinline__ void load(const char* __restrict__ row, const int c) {
        const words* p = reinterpret_cast<const words*>(row) + c;
        v = NT ? __builtin_nontemporal_load(p) : *p;
    }
    // acc += w * piece
    __device__ __forceinline__ void add_to(float (&acc)[N], const float w) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t u = F32 ? v[i] : ((i & 1) ? v[i / 2] & 0xffff0000u : v[i / 2] << 16);
            acc[i] = fmaf(w, __uint_as_float(u), acc[i]);
        }
    }
};

// YF32 / SF32: y_perm / y_shared hold fp32 (else bf16); OF32: out is fp32 (else bf16, RNE).  K: rows a thread has in
// flight at a time, k itself up to 8.
constexpr int COMBINE_MAX_WAVES = 5;
// Elements per thread: 16 bytes of its widest input, twice that for one or two fp32 rows that the cache holds (8 experts top-2, H =
// 6144, 4242 tokens 45.8 -> 38.8 us, H = 4096, 8000 tokens 59.2 -> 55.5; but 16384 tokens, H = 6144, from memory 155 -> 171).
constexpr int combine_elements(const bool fp32, const int k, const bool nt) { return fp32 && (k > 2 || nt) ? 4 : 8; }
template <bool YF32, bool SF32, bool OF32, int K, bool NT>
__global__ __launch_bounds__(COMBINE_MAX_WAVES * 64) void combine_kernel(const char* __restrict__ y_perm, const int32_t* __restrict__ inv_perm,
                                                                         const float* __restrict__ w, const char* __restrict__ y_shared,
                                                                         int k, int H, char* __restrict__ out) {
    constexpr int N = combine_elements(YF32 || SF32, K, NT);
    const int t = blockIdx.x;
    const int c = blockIdx.y * blockDim.x + threadIdx.x;
    if (c >= H / N) return;
    const size_t ybytes = (size_t)H * (YF32 ? 4 : 2);
    const size_t sbytes = (size_t)H * (SF32 ? 4 : 2);
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
    Piece<SF32, N, NT> sh;
    if (y_shared) sh.load(y_shared + (size_t)t * sbytes, c);
    const int32_t* ip = inv_perm + (size_t)t * k;
    const float* wp = w + (size_t)t * k;
    Piece<YF32, N, NT> row[K];
    int j = 0;
    do {   // one pass unless k > 8
#pragma unroll
        for (int i = 0; i < K; ++i) row[i].load(y_perm + (size_t)ip[j + i] * ybytes, c);
#pragma unroll
        for (int i = 0; i < K; ++i) row[i].add_to(acc, wp[j + i]);
        j += K;
    } while (K == 8 && j + K <= k);
    if (K == 8)
        for (; j < k; ++j) {
            row[0].load(y_perm + (size_t)ip[j] * ybytes, c);
            row[0].add_to(acc, wp[j]);
        }
    if (y_shared) sh.add_to(acc, 1.0f);
    if (OF32) {
        float4* o = reinterpret_cast<float4*>(out + (size_t)t * H * 4) + (N / 4) * c;
#pragma unroll
        for (int i = 0; i < N / 4; ++i) o[i] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
    } else {
        typedef __bf16 bf16_n __attribute__((ext_vector_type(N)));
        bf16_n o;
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = (__bf16)acc[i];
        reinterpret_cast<bf16_n*>(out + (size_t)t * H * 2)[c] = o;
    }
}

// One-time weight packing.  in: logical [K, N] bf16 row-major (K = contraction dimension).
// out: the tiled layout the GEMM loads, i.e. the matrix W[n][k] = in[k][n] cut into blocks of
// 16 rows x 32 k (1 KiB), blocks ordered [N/16][K/32]; inside a block, row r (0..15) occupies
// bytes r*64..r*64+63 and its 16-byte piece c (k = 8c..8c+7) sits at slot c ^ ((4 - r/4) & 3).
// Rows keep their logical order.
// One workgroup transposes a 32 k x 32 n patch through LDS.
// N columns exist in `in`; blocks past them (the router pads its expert count to 32) are zero.
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint16_t* __restrict__ in, int K, int N,
                                                          uint16_t* __restrict__ out) {
    __shared__ uint16_t patch[32][34];
    const int kt = blockIdx.x, b = blockIdx.y;      // k sub-tile, 32-row block of W
    const int tid = threadIdx.x;
    for (int i = tid; i < 32 * 32; i += 256) {
        const int kk = i >> 5, nn = i & 31;
        const int n = b * 32 + nn;
        patch[kk][nn] = n < N ? in[(size_t)(kt * 32 + kk) * N + n] : (uint16_t)0;
    }
    __syncthreads();
    if (tid < 128) {
        // 2 groups x 64 pieces; piece id inside the group = r*4 + slot
        const int grp = tid >> 6, pid = tid & 63;
        const int r = pid >> 2, slot = pid & 3;
        const int c = slot ^ block_swizzle(r);
        const int rho = grp * 16 + r;
        const int nloc = rho;
        uint16_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = patch[c * 8 + i][nloc];
        const size_t block = ((size_t)(b * 2 + grp) * (size_t)(K >> 5) + kt) * 512;  // in uint16 units
        uint4 q;
        q.x = v[0] | ((uint32_t)v[1] << 16);
        q.y = v[2] | ((uint32_t)v[3] << 16);
        q.z = v[4] | ((uint32_t)v[5] << 16);
        q.w = v[6] | ((uint32_t)v[7] << 16);
        *reinterpret_cast<uint4*>(out + block + pid * 8) = q;
    }
}

}  // namespace

hipError_t launch_combine(const moe_shape& s, const void* y_perm, const int32_t* inv_perm, const float* w,
                          const void* y_shared, void* out, bool y_fp32, bool shared_fp32, bool out_fp32, hipStream_t st) {
    if (!y_shared) shared_fp32 = y_fp32;   // no rows, so no say in what a thread loads
    if (y_fp32 && !shared_fp32) return hipErrorInvalidValue;   // no caller has fp32 y_perm next to bf16 y_shared
    // Non-temporal loads where the rows exceed the memory-side cache (256 MB): they are read once, most of them from memory
    // (16384 tokens above: 117 us without, 94 with).  Rows that fit are still there from the down GEMM's stores, and
    // the hint costs: 8 experts top-2, H = 4096, fp32, 4096 tokens (134 MB) 28.6 -> 29.9 us.
    const int64_t row_bytes = s.top_k * (y_fp32 ? 4 : 2) + (y_shared ? (shared_fp32 ? 4 : 2) : 0);
    const bool nt = (int64_t)s.T * s.H * row_bytes > ((int64_t)256 << 20);
    // up to five waves to a workgroup, and as many workgroups to a token as its row then takes
    const int per_thread = combine_elements(y_fp32 || shared_fp32, s.top_k, nt);
    const int waves = (s.H / per_thread + 63) / 64, parts = (waves + COMBINE_MAX_WAVES - 1) / COMBINE_MAX_WAVES;
    const dim3 grid((unsigned)s.T, (unsigned)parts), block((unsigned)((waves + parts - 1) / parts * 64));
#define COMBINE_NT(Y, S, O, K, NT)                                                                                        \
    hipLaunchKernelGGL((combine_kernel<Y, S, O, K, NT>), grid, block, 0, st, (const char*)y_perm, inv_perm, w,            \
                       (const char*)y_shared, s.top_k, s.H, (char*)out)
#define COMBINE(Y, S, O, K)                         \
    do {                                            \
        if (nt) COMBINE_NT(Y, S, O, K, true);       \
        else COMBINE_NT(Y, S, O, K, false);         \
    } while (0)
#define COMBINE_K(Y, S, O)                \
    switch (s.top_k) {                    \
        case 1: COMBINE(Y, S, O, 1); break; \
        case 2: COMBINE(Y, S, O, 2); break; \
        case 3: COMBINE(Y, S, O, 3); break; \
        case 4: COMBINE(Y, S, O, 4); break; \
        case 5: COMBINE(Y, S, O, 5); break; \
        case 6: COMBINE(Y, S, O, 6); break; \
        case 7: COMBINE(Y, S, O, 7); break; \
        default: COMBINE(Y, S, O, 8); break; \
    }
#define COMBINE_O(Y, S)                      \
    do {                                     \
        if (out_fp32) COMBINE_K(Y, S, true)  \
        else COMBINE_K(Y, S, false)          \
    } while (0)
    if (y_fp32 && shared_fp32) COMBINE_O(true, true);
    else if (shared_fp32) COMBINE_O(false, true);
    else COMBINE_O(false, false);
#undef COMBINE_O
#undef COMBINE_K
#undef COMBINE
#undef COMBINE_NT
    return hipGetLastError();
}

hipError_t launch_pack_weight(const void* in, int rows, int cols, int cols_padded, void* out, hipStream_t st) {
    const dim3 grid(rows / 32, cols_padded / 32);   // rows = K, cols = N
    hipLaunchKernelGGL(pack_weight_kernel, grid, dim3(256), 0, st, (const uint16_t*)in, rows, cols, (uint16_t*)out);
    return hipGetLastError();
}

}  // namespace moe
