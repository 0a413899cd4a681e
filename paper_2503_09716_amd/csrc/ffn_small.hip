// Grouped FFN GEMMs of small batches: few rows per group, so what a launch does is read weights.
//
// The tile routine of ffn_gemm.hip gives a workgroup 256 rows of W and a whole CU.  With few groups
// that leaves most of the chip idle (one token on 64 experts top-6 with two shared ones: 88 and 56
// tiles for 256 CUs), and a CU by itself fills its LDS at about 44 GB/s.  Here the unit of work is
// one wavefront: 16 or 32 output columns of one group (gate/up: as many rows of both matrices) over the
// whole of K, for up to 64 rows of X.  W goes straight from memory into registers - a 16 x 32 block of
// the packed layout is one 1 KiB load, already in operand order up to a lane permutation - through
// a ring of RING sub-tiles per wave (about 32 KiB in flight), with no LDS and no barrier.  X is read the
// same way; its rows are few and come from L2.  A group of up to 64 rows reads its W once; in a layer that no
// cache can hold those loads are non-temporal, which is worth a tenth (8x7B, 8 tokens: gate/up 297 -> 267 us,
// down 146 -> 128 = 7.3 TB/s; 64 experts, 16 tokens: 107 -> 98, 53 -> 47).  A taller group reads it once per 64
// rows, and the hint then costs more than it gives (4 experts of 4, H = 8192, F = 1408, 100 tokens: gate/up
// 92 us without, 115 with it).
//
// Every output element is one chain of v_mfma_f32_16x16x32_bf16 over K in ascending order with the
// operands in the same roles as in the tile routine, so both give the same bits.
#include "common.h"

namespace moe {
namespace {

// Global-memory pointers, said so: a pointer read from a table is generic to the compiler, and after
// generic (flat) loads it waits for every load in flight.
typedef const __attribute__((address_space(1))) char* gchar_t;
typedef const __attribute__((address_space(1))) bf16x8* gfrag_t;

constexpr int SMALL_ROWS = 64;   // rows of X per wave at most: an m-tile of up to 128 rows is two units

// One unit: rows r0 .. r0 + 16 * XB - 1 of tile d (nrows of the tile are valid), columns n0 .. n0 + 16 * NB - 1.
// ROUTER: the gate GEMM, K piece d.group of one packed matrix, fp32 partial logits.
// NT: W loads are non-temporal.
template <bool GATED, int NB, int XB, int RING, bool NT, bool ROUTER = false>
__device__ __forceinline__ void small_unit(const GemmArgs& p, const TileDesc d, const int r0, const int n0, const int lane) {
    constexpr int WQ = GATED ? 2 * NB : NB;   // W blocks per sub-tile
    const int rl = lane & 15, g = lane >> 4;
    const bool shared = !ROUTER && d.srow >= 0;
    const int nseg = !GATED && shared ? p.nseg_shared : 1;
    const int KT = p.K >> 5;
    const bool a_tiled = !ROUTER && ((shared ? p.a_tiled >> 1 : p.a_tiled) & 1) != 0;
    const uint32_t xstep = a_tiled ? 1024 : 64;
    const size_t a_seg_stride = (size_t)p.t_pad * (size_t)p.K * 2;
    // per-lane byte offsets: row rl of each block, logical 16-byte piece g
    uint32_t xoff[XB];
#pragma unroll
    for (int i = 0; i < XB; ++i) {
        int grow = d.row0 + min(r0 + i * 16 + rl, d.nrows - 1);   // padded rows re-read the last valid row
        if (!a_tiled) {
            if (!ROUTER && !shared && p.row_token) grow = p.row_token[grow];
            xoff[i] = (uint32_t)grow * (uint32_t)p.lda_bytes + (uint32_t)(g * 16);
        } else {
            const int rr = grow & 15;
            xoff[i] = (uint32_t)(grow >> 4) * (uint32_t)(p.kt_a * 1024) + (uint32_t)(rr * 64 + ((g ^ block_swizzle(rr)) << 4));
        }
    }
    const uint32_t woff = (uint32_t)(n0 >> 4) * (uint32_t)(p.kt_w * 1024) + (uint32_t)(rl * 64 + ((g ^ block_swizzle(rl)) << 4));

    f32x4 acc[WQ][XB];
#pragma unroll
    for (int j = 0; j < WQ; ++j)
#pragma unroll
        for (int i = 0; i < XB; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wf[RING][WQ], xf[RING][XB];

    gchar_t xb = (gchar_t)(shared ? p.a_shared : p.a_routed) + (ROUTER ? (size_t)d.group * (size_t)p.K * 2 : 0);
    gchar_t wa = ROUTER ? (gchar_t)p.w_uniform + (size_t)d.group * (size_t)p.w_uniform_stride : (gchar_t)p.w_a[d.group];
    gchar_t const wb = GATED ? (gchar_t)p.w_b[d.group] : (gchar_t)nullptr;
    auto load = [&](const int u, gchar_t x, gchar_t w, const int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < WQ; ++j) {
            gchar_t base = GATED && j >= NB ? wb : w;
            const uint32_t off = woff + (uint32_t)((GATED && j >= NB ? j - NB : j) * p.kt_w + ks) * 1024u;
            wf[u][j] = NT ? __builtin_nontemporal_load((gfrag_t)(base + off)) : *(gfrag_t)(base + off);
        }
#pragma unroll
        for (int i = 0; i < XB; ++i) xf[u][i] = *(gfrag_t)(x + (xoff[i] + (uint32_t)ks * xstep));
    };
    auto multiply = [&](const int u) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < WQ; ++j)
#pragma unroll
            for (int i = 0; i < XB; ++i)
                acc[j][i] = GATED ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u][j], xf[u][i], acc[j][i], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[u][i], wf[u][j], acc[j][i], 0, 0, 0);
    };
    // Sub-tile t sits in ring place t % RING (counted from the segment's start), and a place is
    // refilled right after its last use.  No load in the loop over K is inside a branch (the compiler would have to
    // wait for all loads behind it): past the end of K the places take the first sub-tiles of the next
    // segment, or re-read the last sub-tile.  (The branch after it, once per segment, only loads where there is a next one.)
#pragma unroll
    for (int u = 0; u < RING; ++u) load(u, xb, wa, min(u, KT - 1));
    for (int seg = 0; seg < nseg; ++seg) {
        const bool more = seg + 1 < nseg;
        gchar_t const xn = more ? xb + a_seg_stride : xb;
        gchar_t const wn = more ? (gchar_t)p.w_a[d.group + seg + 1] : wa;
        int t = 0;
        for (; t + 2 * RING <= KT; t += RING) {
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                multiply(u);
                load(u, xb, wa, t + RING + u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < RING; ++u) {
            if (t + u < KT) multiply(u);
            const int ks = t + RING + u;
            const bool in = ks < KT;
            load(u, in ? xb : xn, in ? wa : wn, in ? ks : (more ? min(u, KT - 1) : KT - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < RING; ++u) {
            if (t + RING + u < KT) {
                multiply(u);
                if (more) load(u, xn, wn, min(u, KT - 1));
            }
        }
        xb = xn;
        wa = wn;
    }

    if (GATED) {
        // lane: output row rl of X block i, columns 4g .. 4g+3 of gate block j; h is written in its tiled layout
        const int orow_base = (shared ? d.srow : 0) + d.row0;
        char* const out = shared ? p.out_shared : p.out_routed;
#pragma unroll
        for (int i = 0; i < XB; ++i) {
            const int r = r0 + i * 16 + rl;
            if (r >= d.nrows) continue;
            const int ro = orow_base + r, rr = ro & 15, sw = block_swizzle(rr);
            char* hrow = out + ((size_t)(ro >> 4) * (size_t)(p.N >> 5)) * 1024 + rr * 64;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int col = n0 + j * 16 + g * 4;
                bf16x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float gv = acc[j][i][q], uv = acc[NB + j][i][q];
                    o[q] = (__bf16)(gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv)) * uv);
                }
                *reinterpret_cast<bf16x4*>(hrow + (size_t)(col >> 5) * 1024 + ((((col & 31) >> 3) ^ sw) << 4) + (col & 7) * 2) = o;
            }
        }
    } else {
        // lane: output column rl of W block j, rows 4g .. 4g+3 of X block i
        const bool f32 = ROUTER || ((shared ? p.out_fp32 >> 1 : p.out_fp32) & 1) != 0;
        char* const out = shared ? p.out_shared : p.out_routed;
#pragma unroll
        for (int i = 0; i < XB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + i * 16 + g * 4 + q;
                if (r >= d.nrows) continue;
                const size_t at = (size_t)((ROUTER ? d.group * p.split_rows : 0) + d.row0 + r) * (size_t)p.N + (size_t)(n0 + rl);
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if (f32) reinterpret_cast<float*>(out)[at + j * 16] = acc[j][i][q];
                    else reinterpret_cast<__bf16*>(out)[at + j * 16] = (__bf16)acc[j][i][q];
                }
            }
    }
}

// Units in the order: columns fastest, then the 64-row parts of an m-tile (`halves` of them side by
// side; a unit takes every halves-th part, whatever the tile's height), then m-tiles.
template <bool GATED, int NB, bool NT>
__global__ __launch_bounds__(64, 2) void ffn_small_kernel(const GemmArgs p, const int halves) {
    const int lane = threadIdx.x;
    const int per = p.n_tiles * halves;
    const int mt = blockIdx.x / per;
    if (mt >= (GATED ? p.plan->n_gate_up : p.plan->n_down)) return;
    const int rem = blockIdx.x - mt * per, half = rem / p.n_tiles;
    TileDesc d = p.descs[mt];
    d.nrows &= TILE_ROWS_MASK;
    const int n0 = (rem - half * p.n_tiles) * 16 * NB;
    for (int r0 = half * SMALL_ROWS; r0 < d.nrows; r0 += halves * SMALL_ROWS) {
        const int blocks = (min(d.nrows - r0, SMALL_ROWS) + 15) >> 4;   // wave-uniform
        if (blocks > 2) small_unit<GATED, NB, 4, GATED ? 4 : (NB == 2 ? 5 : 6), NT>(p, d, r0, n0, lane);
        else if (blocks > 1) small_unit<GATED, NB, 2, GATED ? 6 : (NB == 2 ? 7 : 8), NT>(p, d, r0, n0, lane);
        else small_unit<GATED, NB, 1, GATED ? 8 : (NB == 2 ? 8 : 16), NT>(p, d, r0, n0, lane);
    }
}

// Router GEMM of a small batch: one wave per 16 tokens, 16 experts and K piece.  The tile routine has one
// workgroup per K piece and 128 tokens, four in all for a small batch, each of which reads a quarter of
// the gate matrix by itself.
__global__ __launch_bounds__(64, 2) void route_small_kernel(const GemmArgs p) {
    const int cols = p.N >> 4, rows = (p.T + 15) >> 4;
    const int nb = blockIdx.x % cols, m = (blockIdx.x / cols) % rows, s = blockIdx.x / (cols * rows);
    TileDesc d;
    d.group = s;
    d.row0 = m * 16;
    d.nrows = min(16, p.T - d.row0);
    d.srow = -1;
    small_unit<false, 1, 1, 16, false, true>(p, d, 0, nb * 16, threadIdx.x);
}

}  // namespace

hipError_t launch_route_small(const GemmArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(route_small_kernel, dim3((unsigned)((a.N / 16) * ((a.T + 15) / 16) * a.uniform_splits)), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_ffn_small(bool gated, const GemmArgs& a, int col_blocks, int halves, bool nt, hipStream_t st) {
    // one wave per workgroup: four to a workgroup leave CUs idle at the sizes this is for (1 token: 22 -> 31 us)
    const dim3 grid((unsigned)a.max_mtiles * (unsigned)(a.n_tiles * halves)), block(64);
#define SMALL(G_, NB_)                                                                                   \
    do {                                                                                                 \
        if (nt) hipLaunchKernelGGL((ffn_small_kernel<G_, NB_, true>), grid, block, 0, st, a, halves);    \
        else hipLaunchKernelGGL((ffn_small_kernel<G_, NB_, false>), grid, block, 0, st, a, halves);      \
    } while (0)
    if (gated) SMALL(true, 2);
    else if (col_blocks == 2) SMALL(false, 2);
    else SMALL(false, 1);
#undef SMALL
    return hipGetLastError();
}

}  // namespace moe
