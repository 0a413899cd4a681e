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
#include "topk.h"

namespace moe {
namespace {

// Global-memory pointers, said so: a pointer read from a table is generic to the compiler, and after
// generic (flat) loads it waits for every load in flight.
typedef const __attribute__((address_space(1))) char* gchar_t;
typedef const __attribute__((address_space(1))) bf16x8* gfrag_t;

constexpr int SMALL_ROWS = 64;   // rows of X per wave at most: an m-tile of up to 128 rows is two units

// Where a unit's W comes from: rows n0 .. of expert `group`'s matrices, per lane row lane % 16 of a block, logical piece lane / 16.
template <bool GATED, int NB>
struct Panel {
    static constexpr int WQ = GATED ? 2 * NB : NB;   // W blocks per sub-tile
    gchar_t a, b;
    uint32_t off;
    __device__ __forceinline__ Panel(const GemmArgs& p, gchar_t wa, gchar_t wb, const int n0, const int lane) : a(wa), b(wb) {
        const int rl = lane & 15, g = lane >> 4;
        off = (uint32_t)(n0 >> 4) * (uint32_t)(p.kt_w * 1024) + (uint32_t)(rl * 64 + ((g ^ block_swizzle(rl)) << 4));
    }
    __device__ __forceinline__ Panel(const GemmArgs& p, const int group, const int n0, const int lane)
        : Panel(p, (gchar_t)p.w_a[group], GATED ? (gchar_t)p.w_b[group] : (gchar_t)nullptr, n0, lane) {}
    // sub-tile ks
    template <bool NT>
    __device__ __forceinline__ void load(const GemmArgs& p, const int ks, bf16x8 (&f)[WQ]) const {
#pragma unroll
        for (int j = 0; j < WQ; ++j) {
            gchar_t base = GATED && j >= NB ? b : a;
            const uint32_t at = off + (uint32_t)((GATED && j >= NB ? j - NB : j) * p.kt_w + ks) * 1024u;
            f[j] = NT ? __builtin_nontemporal_load((gfrag_t)(base + at)) : *(gfrag_t)(base + at);
        }
    }
};

// The first sub-tiles of a unit's W, asked for before the unit's rows are known: their latency passes while the rows are looked up.
// Only where the candidate is a pair's expert (no more pairs than experts), which has rows: the matrices of an expert without rows are
// not touched, they need not be resident.
// Layers of one token, us: 35.0 -> 33.9 (64 experts, F = 1408), 116.7 -> 114.9 (8 experts, F = 14336).  Not in the gate/up GEMM
// of more than 16 tokens, whose registers are full (12.7 -> 13.2), nor where the expert has to be searched first (no change).
constexpr int EARLY = 4;
template <bool GATED, int NB>
struct EarlyW {
    bf16x8 f[EARLY][Panel<GATED, NB>::WQ];
    template <bool NT>
    __device__ __forceinline__ void ask(const GemmArgs& p, const int group, const int n0, const int lane) {
        const Panel<GATED, NB> w(p, group, n0, lane);
#pragma unroll
        for (int u = 0; u < EARLY; ++u) w.template load<NT>(p, min(u, (p.K >> 5) - 1), f[u]);
    }
};

// One unit: rows r0 .. r0 + 16 * XB - 1 of tile d (nrows of the tile are valid), columns n0 .. n0 + 16 * NB - 1.
// ROUTER: the gate GEMM, K piece d.group of one packed matrix, fp32 partial logits.
// NT: W loads are non-temporal.  tokens: row r of a routed tile is token tokens[r] (LDS) instead of row_token's.
template <bool GATED, int NB, int XB, int RING, bool NT, bool ROUTER = false>
__device__ __forceinline__ void small_unit(const GemmArgs& p, const TileDesc d, const int r0, const int n0, const int lane,
                                           const int* tokens = nullptr, const EarlyW<GATED, NB>* early = nullptr) {
    constexpr int WQ = Panel<GATED, NB>::WQ;
    static_assert(RING >= EARLY, "early sub-tiles fill the first places of the ring");
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
            if (!ROUTER && !shared && tokens) grow = tokens[grow - d.row0];
            else if (!ROUTER && !shared && p.row_token) grow = p.row_token[grow];
            xoff[i] = (uint32_t)grow * (uint32_t)p.lda_bytes + (uint32_t)(g * 16);
        } else {
            const int rr = grow & 15;
            xoff[i] = (uint32_t)(grow >> 4) * (uint32_t)(p.kt_a * 1024) + (uint32_t)(rr * 64 + ((g ^ block_swizzle(rr)) << 4));
        }
    }
    f32x4 acc[WQ][XB];
#pragma unroll
    for (int j = 0; j < WQ; ++j)
#pragma unroll
        for (int i = 0; i < XB; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wf[RING][WQ], xf[RING][XB];

    gchar_t xb = (gchar_t)(shared ? p.a_shared : p.a_routed) + (ROUTER ? (size_t)d.group * (size_t)p.K * 2 : 0);
    const gchar_t w0 = ROUTER ? (gchar_t)p.w_uniform + (size_t)d.group * (size_t)p.w_uniform_stride : (gchar_t)p.w_a[d.group];
    Panel<GATED, NB> wa(p, w0, GATED ? (gchar_t)p.w_b[d.group] : (gchar_t)nullptr, n0, lane);
    auto load_x = [&](const int u, gchar_t x, const int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < XB; ++i) xf[u][i] = *(gfrag_t)(x + (xoff[i] + (uint32_t)ks * xstep));
    };
    auto load = [&](const int u, gchar_t x, const Panel<GATED, NB>& w, const int ks) __attribute__((always_inline)) {
        w.template load<NT>(p, ks, wf[u]);
        load_x(u, x, ks);
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
    for (int u = 0; u < RING; ++u) {
        if (early && u < EARLY) {
#pragma unroll
            for (int j = 0; j < WQ; ++j) wf[u][j] = early->f[u][j];
            load_x(u, xb, min(u, KT - 1));
        } else {
            load(u, xb, wa, min(u, KT - 1));
        }
    }
    for (int seg = 0; seg < nseg; ++seg) {
        const bool more = seg + 1 < nseg;
        gchar_t const xn = more ? xb + a_seg_stride : xb;
        Panel<GATED, NB> wn = wa;
        if (more) wn.a = (gchar_t)p.w_a[d.group + seg + 1];
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

// Up to 64 rows of tile d from row r0 on, columns n0 ..
template <bool GATED, int NB, bool NT>
__device__ __forceinline__ void small_block(const GemmArgs& p, const TileDesc& d, const int r0, const int n0, const int lane, const int* tokens = nullptr,
                                            const EarlyW<GATED, NB>* early = nullptr) {
    const int blocks = (min(d.nrows - r0, SMALL_ROWS) + 15) >> 4;   // wave-uniform
    if (blocks > 2) small_unit<GATED, NB, 4, GATED ? 4 : (NB == 2 ? 5 : 6), NT>(p, d, r0, n0, lane, tokens, early);
    else if (blocks > 1) small_unit<GATED, NB, 2, GATED ? 6 : (NB == 2 ? 7 : 8), NT>(p, d, r0, n0, lane, tokens, early);
    else if (blocks > 0) small_unit<GATED, NB, 1, GATED ? 8 : (NB == 2 ? 8 : 16), NT>(p, d, r0, n0, lane, tokens, early);
}

// Part `part` of `parts` of tile d: every parts-th 64 rows
template <bool GATED, int NB, bool NT>
__device__ __forceinline__ void small_rows(const GemmArgs& p, const TileDesc& d, const int part, const int parts, const int n0, const int lane) {
    for (int r0 = part * SMALL_ROWS; r0 < d.nrows; r0 += parts * SMALL_ROWS) small_block<GATED, NB, NT>(p, d, r0, n0, lane);
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
    small_rows<GATED, NB, NT>(p, d, half, halves, (rem - half * p.n_tiles) * 16 * NB, lane);
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

// ---- layers of few pairs: up to 16 tokens, or up to 256 in small layers ---------------------------------------
// What a wave needs to know of the routing - its expert's tokens and where their rows begin - it reads off topk_idx itself
// (at most 1024 pairs, a vote per 64; in the down GEMM mostly off expert_offsets).  So no launch stands between the selection and the gate/up GEMM: expert_offsets and
// inv_perm are written by one wave of that GEMM's launch.  Up to 16 tokens every group is one block of 16 rows, and with more
// than 16 experts the shared ones can run ahead (launch_decode says where): their gate/up GEMM next to the top-k, whose
// launch leaves the memory idle, and their down GEMM, the longest walk of all, next to the routed gate/up GEMM.  (The first
// part of that next to the router GEMM instead: 2 us slower.)  Same bits as the launches by list.  Layer, us: 64 experts
// top-6 + 2 shared, F = 1408, 1 token 42.2 -> 35.7, 4: 85 -> 79, 16: 167 -> 158; 160 experts, 1: 82 -> 74, 16: 583 -> 568; 8
// experts top-2, F = 14336, 1: 125 -> 116, 16: 441 -> 430; H = 512, F = 1024, 8 tokens 23 -> 17, 40: 24.7 -> 21.1,
// 256: 31.1 -> 26.5.
struct Group {
    int expert, row0, rows;
};
// Orders a wave's LDS writes and reads (one wave to a workgroup; a barrier would wait for the loads in flight).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// The pairs v (of index base + lane) that have expert e: their tokens (unless nullptr) and number, and the number of those with lower ones.
template <int MAX>
__device__ __forceinline__ void count_pairs(const DecodeArgs& a, const int e, const int v, const uint64_t eq, const int base, const int lane, int* tokens,
                                            int& n, int& before) {
    if (eq) {
        if (tokens) {
            const int rank = n + __popcll(eq & ((1ull << lane) - 1));
            if (v == e && rank < MAX) tokens[rank] = (int)((uint32_t)(base + lane) * a.inv_k >> 16);
        }
        n += __popcll(eq);
    }
    before += __popcll(__ballot(v < e));
}
// Candidate c of the routed groups: expert c, or with fewer pairs than experts the expert of pair c, of which the first
// pair that has it is taken.  False: no rows.
// MAX: tokens at most; the pairs come 64 * CHUNKS at a time, all loads of which are in flight together.
// ask(expert) comes between the first loads of the pairs and their use (EarlyW).
template <int MAX, class Ask>
__device__ __forceinline__ bool candidate_group(const DecodeArgs& a, const int c, const int lane, Group& g, int* tokens, Ask ask) {
    constexpr int CHUNKS = MAX <= 16 ? 1 : 8;   // (few pairs: more code costs more than loads in turn, 1 token 0.8 us)
    const bool by_pair = a.pairs <= a.E;
    const int e = __builtin_amdgcn_readfirstlane(by_pair ? a.topk_idx[c] : c);
    int n = 0, before = 0, v[CHUNKS];
    auto get = [&](const int base) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) v[u] = a.topk_idx[min(base + u * 64 + lane, a.pairs - 1)];
    };
    // false: an earlier pair has the expert
    auto count = [&](const int base) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            if (base + u * 64 + lane >= a.pairs) v[u] = 0x7fffffff;
            const uint64_t eq = __ballot(v[u] == e);
            if (by_pair && n == 0 && eq && base + u * 64 + __builtin_ctzll(eq) != c) return false;
            count_pairs<MAX>(a, e, v[u], eq, base + u * 64, lane, tokens, n, before);
        }
        return true;
    };
    get(0);
    ask(e);
    if (!count(0)) return false;
    for (int base = 64 * CHUNKS; base < a.pairs; base += 64 * CHUNKS) {
        get(base);
        if (!count(base)) return false;
    }
    wave_lds_order();
    g.expert = e;
    g.row0 = before;
    g.rows = min(n, MAX);   // a token has an expert once
    return n > 0;
}
// The c-th expert that has rows, of up to 256 pairs, so that the waves without work are the launch's last.  Spread
// between the others (candidate_group) they leave some CUs a wave more than others, which counts where a launch fills the chip about once (8
// experts top-2, H = 6144, F = 16384, 3 tokens that pick 4 experts: gate/up 262 -> 239 us, 4 tokens, 6 experts 374 -> 352, 64 experts
// top-6, 10 tokens 90 -> 85), and not in a small layer, whose waves take longer to find it (256 tokens 26.8 -> 29.4).
__device__ __forceinline__ bool active_group(const DecodeArgs& a, const int c, const int lane, Group& g, int* tokens) {
    __shared__ uint32_t present[8];   // bit e: expert e has rows
    int v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = u * 64 + lane < a.pairs ? a.topk_idx[u * 64 + lane] : 0x7fffffff;
    if (lane < 8) present[lane] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u * 64 + lane < a.pairs) atomicOr(&present[v[u] >> 5], 1u << (v[u] & 31));
    __syncthreads();
    int left = c, word = -1;
    uint32_t bits = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const uint32_t m = present[w];
        if (word < 0 && left < __popc(m)) { word = w; bits = m; }
        if (word < 0) left -= __popc(m);
    }
    if (word < 0) return false;
    const uint64_t hit = __ballot(lane < 32 && (bits >> lane & 1) && __popc(bits & ((1u << lane) - 1)) == left);
    const int e = __builtin_amdgcn_readfirstlane(word * 32 + __builtin_ctzll(hit));
    int n = 0, before = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u * 64 < a.pairs) count_pairs<16>(a, e, v[u], __ballot(v[u] == e), u * 64, lane, tokens, n, before);
    wave_lds_order();
    g.expert = e;
    g.row0 = before;
    g.rows = min(n, 16);
    return true;
}
// Down GEMM, more pairs than experts: expert c's rows off the offsets that decode_index wrote in the gate/up GEMM's launch.  They are there
// after one load, so W is asked for once it is known that the expert has rows.  Layer against counting the pairs again behind an EarlyW of every
// expert: H = 512, F = 1024, 8 experts, 128 tokens 20.4 -> 20.1 us, 256: 23.9 -> 23.6, 6 experts, H = 1280, F = 896, 48 tokens 20.9 -> 20.5; up to
// 16 tokens 0.2 us more for the down GEMM (and 0.6 for the gate/up GEMM without EarlyW).
__device__ __forceinline__ bool indexed_group(const GemmArgs& down, const DecodeArgs& a, const int c, Group& g) {
    const int row0 = a.offsets[c], end = a.offsets[c + 1];
    const bool there = down.w_a[c] != nullptr;   // always: puts the load of the matrix's address next to the two above
    g.expert = c;
    g.row0 = __builtin_amdgcn_readfirstlane(row0);
    g.rows = __builtin_amdgcn_readfirstlane(end - row0);
    return (g.rows > 0) & there;
}
// expert_offsets and inv_perm, by one wave (E <= 256, at most 64 * CHUNKS pairs): what the combine and moe_layer_views read.  perm
// and row_token have no reader in these layers.
template <int CHUNKS>
__device__ __forceinline__ void decode_index(const DecodeArgs& a, const int lane) {
    __shared__ int cursor[256];
    __shared__ unsigned long long mask[256];
    int v[CHUNKS];
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) v[u] = u * 64 + lane < a.pairs ? a.topk_idx[u * 64 + lane] : -1;
    for (int e = lane; e < 256; e += 64) { cursor[e] = 0; mask[e] = 0; }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u)
        if (v[u] >= 0) atomicAdd(&cursor[v[u]], 1);
    __syncthreads();
    int count[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) { count[i] = cursor[4 * lane + i]; sum += count[i]; }
    int before = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(before, d, 64);
        if (lane >= d) before += t;
    }
    before -= sum;
    int start[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = 4 * lane + i;
        cursor[e] = before;
        start[i] = before;
        before += count[i];
    }
    __syncthreads();
    int slot[CHUNKS];   // written at the end: a barrier waits for the stores before it
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
        if (u * 64 >= a.pairs) break;
        const int e = max(v[u], 0);
        if (v[u] >= 0) atomicOr(&mask[e], 1ull << lane);
        __syncthreads();
        const unsigned long long m = mask[e];
        const int rank = __popcll(m & ((1ull << lane) - 1));
        slot[u] = cursor[e] + rank;
        __syncthreads();
        if (v[u] >= 0 && rank == 0) { cursor[e] += __popcll(m); mask[e] = 0; }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (4 * lane + i < a.E) a.offsets[4 * lane + i] = start[i];
    if (lane == 0) a.offsets[a.E] = a.pairs;
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
        const int p = u * 64 + lane;
        if (v[u] < 0) continue;
        a.inv_perm[p] = slot[u];
    }
}

__device__ __forceinline__ TileDesc shared_tile(const DecodeArgs& a, const GemmArgs& p, const int s) { return {a.E + s, 0, p.T, s * p.t_pad}; }

// Gate/up units of 16 columns (UB = 1) while the weights come from memory: twice the waves, and so bytes in flight, of units of 32 (64
// experts, 1 token 38.9 -> 35.7 us, 160: 83.9 -> 74.5, 16 tokens 159 -> 155); a layer that the cache holds is faster with 32 (H =
// 512, F = 1024, 16 tokens 17.3 us, 18.1 with 16), and so are those above the cache
// size whose walk along K is no longer than it takes a wave to find its group and fill its ring (H < 768) or whose units of 32 fill
// the chip, two to a SIMD, about once, so that 16 add half a round (550 layers of 1 to 16 tokens: 16 columns take 1.05 and 1.03 of
// the time of 32 there, 1.10 and 1.09 at most, elsewhere 0.98).
template <int UB, bool NT>
__device__ __forceinline__ void up_unit(const GemmArgs& up, const TileDesc& d, const int unit, const int lane, const int* tokens = nullptr,
                                        const EarlyW<true, UB>* early = nullptr) {
    small_unit<true, UB, 1, 16 / UB, NT>(up, d, 0, unit * 16 * UB, lane, tokens, early);
}
// Gate/up unit `unit` of all shared experts'.
template <int UB, bool NT>
__device__ __forceinline__ void shared_up_unit(const GemmArgs& up, const DecodeArgs& a, const int unit, const int lane) {
    const int s = unit / up.n_tiles;
    up_unit<UB, NT>(up, shared_tile(a, up, s), unit - s * up.n_tiles, lane);
}

// Top-k of four tokens per workgroup, then the shared experts' gate/up units.
template <int NB, int UB, bool NT>
__global__ __launch_bounds__(64, 2) void decode_topk_kernel(const GemmArgs up, const DecodeArgs a) {
    const int lane = threadIdx.x, quads = (up.T + 3) >> 2, b = blockIdx.x;
    if (b < quads) topk_row16<NB>(a.partial, a.splits, up.T, a.ep, a.E, a.k, a.bias, a.renorm, a.scale, b, lane, a.topk_idx, a.topk_w, nullptr);
    else shared_up_unit<UB, NT>(up, a, b - quads, lane);
}

// Workgroup 0: expert_offsets and inv_perm.  Then the shared experts' down units (early: their gate/up units are done) or gate/up units,
// then the routed gate/up units.
template <int UB, bool NT>
__global__ __launch_bounds__(64, 2) void decode_up_kernel(const GemmArgs up, const GemmArgs down, const DecodeArgs a, const bool early) {
    __shared__ int tokens[16];
    const int lane = threadIdx.x;
    if (blockIdx.x == 0) {
        decode_index<4>(a, lane);
        return;
    }
    int b = blockIdx.x - 1;
    if (early) {
        if (b < down.n_tiles) {
            small_unit<false, 1, 1, 16, NT>(down, shared_tile(a, down, 0), 0, b * 16, lane);
            return;
        }
        b -= down.n_tiles;
    } else if (b < a.Ns * up.n_tiles) {
        shared_up_unit<UB, NT>(up, a, b, lane);
        return;
    } else {
        b -= a.Ns * up.n_tiles;
    }
    const int c = b / up.n_tiles, unit = b - c * up.n_tiles;
    Group g;
    if (NT ? a.pairs != a.k : a.pairs > a.E) {   // one token: every pair another expert
        if (NT ? active_group(a, c, lane, g, tokens) : candidate_group<16>(a, c, lane, g, tokens, [](int) {}))
            up_unit<UB, NT>(up, {g.expert, g.row0, g.rows, -1}, unit, lane, tokens);
        return;
    }
    EarlyW<true, UB> w;
    if (!candidate_group<16>(a, c, lane, g, tokens, [&](const int e) { w.template ask<NT>(up, e, unit * 16 * UB, lane); })) return;
    up_unit<UB, NT>(up, {g.expert, g.row0, g.rows, -1}, unit, lane, tokens, &w);
}

// The shared experts' down units (unless early), then the routed ones.
template <bool NT>
__global__ __launch_bounds__(64, 2) void decode_down_kernel(const GemmArgs down, const DecodeArgs a, const bool early) {
    const int lane = threadIdx.x;
    int b = blockIdx.x;
    if (!early && a.Ns > 0) {
        if (b < down.n_tiles) {
            small_unit<false, 1, 1, 16, NT>(down, shared_tile(a, down, 0), 0, b * 16, lane);
            return;
        }
        b -= down.n_tiles;
    }
    const int c = b / down.n_tiles, n0 = (b - c * down.n_tiles) * 16;
    Group g;
    if (NT ? a.pairs != a.k : a.pairs > a.E) {
        if (NT ? active_group(a, c, lane, g, nullptr) : indexed_group(down, a, c, g)) small_unit<false, 1, 1, 16, NT>(down, {g.expert, g.row0, g.rows, -1}, 0, n0, lane);
        return;
    }
    EarlyW<false, 1> w;
    if (!candidate_group<16>(a, c, lane, g, nullptr, [&](const int e) { w.template ask<NT>(down, e, n0, lane); })) return;
    small_unit<false, 1, 1, 16, NT>(down, {g.expert, g.row0, g.rows, -1}, 0, n0, lane, nullptr, &w);
}

// More than 16 tokens: the same with `parts` waves for every 64 rows of a group.  Workgroup 0: expert_offsets and inv_perm; then all
// groups' first 64 rows (shared experts first), their second, and so on.  (Parts of a group next to each other: most are empty and
// the dispatch lines up the others on the same CUs, H = 512, F = 1024, 8 experts, 256 tokens, four parts: gate/up 9 -> 19 us.)
constexpr int WIDE_TOKENS = 256;
template <bool NT>
__global__ __launch_bounds__(64, 2) void decode_wide_up_kernel(const GemmArgs up, const DecodeArgs a, const int parts, const int groups) {
    __shared__ int tokens[WIDE_TOKENS];
    const int lane = threadIdx.x;
    if (blockIdx.x == 0) {
        decode_index<16>(a, lane);
        return;
    }
    const int b = blockIdx.x - 1, unit = b % up.n_tiles, q = b / up.n_tiles, part = q / groups, c = q - part * groups - a.Ns;
    if (c < 0) {
        small_block<true, 2, NT>(up, shared_tile(a, up, c + a.Ns), part * SMALL_ROWS, unit * 32, lane);
        return;
    }
    Group g;
    if (candidate_group<WIDE_TOKENS>(a, c, lane, g, tokens, [](int) {}))
        small_block<true, 2, NT>(up, {g.expert, g.row0, g.rows, -1}, part * SMALL_ROWS, unit * 32, lane, tokens);
}
template <int NB, bool NT>
__global__ __launch_bounds__(64, 2) void decode_wide_down_kernel(const GemmArgs down, const DecodeArgs a, const int parts, const int groups) {
    const int lane = threadIdx.x, b = blockIdx.x, unit = b % down.n_tiles, q = b / down.n_tiles, part = q / groups, c = q - part * groups - (a.Ns > 0);
    if (c < 0) {
        small_block<false, NB, NT>(down, shared_tile(a, down, 0), part * SMALL_ROWS, unit * 16 * NB, lane);
        return;
    }
    Group g;
    if (a.pairs > a.E) {
        if (indexed_group(down, a, c, g))
            small_block<false, NB, NT>(down, {g.expert, g.row0, g.rows, -1}, part * SMALL_ROWS, unit * 16 * NB, lane);
        return;
    }
    EarlyW<false, NB> w;
    if (!candidate_group<WIDE_TOKENS>(a, c, lane, g, nullptr, [&](const int e) { w.template ask<NT>(down, e, unit * 16 * NB, lane); })) return;
    small_block<false, NB, NT>(down, {g.expert, g.row0, g.rows, -1}, part * SMALL_ROWS, unit * 16 * NB, lane, nullptr, &w);
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

namespace {
template <int UB, bool NT>
hipError_t launch_decode_units(const DecodeStep step, GemmArgs up, const GemmArgs& down, const DecodeArgs& a, const bool early, hipStream_t st) {
    const int candidates = a.pairs < a.E ? a.pairs : a.E;
    const dim3 block(64);
    up.n_tiles = up.N / (16 * UB);
    const int shared_units = a.Ns * up.n_tiles;
#define DECODE(grid_, K_, ...) hipLaunchKernelGGL((K_), dim3((unsigned)(grid_)), block, 0, st, __VA_ARGS__)
    if (step == DECODE_TOPK && a.partial) {
        const int grid = (up.T + 3) / 4 + (early ? shared_units : 0);
        if (a.E <= 64) DECODE(grid, (decode_topk_kernel<1, UB, NT>), up, a);
        else if (a.E <= 128) DECODE(grid, (decode_topk_kernel<2, UB, NT>), up, a);
        else if (a.E <= 192) DECODE(grid, (decode_topk_kernel<3, UB, NT>), up, a);
        else DECODE(grid, (decode_topk_kernel<4, UB, NT>), up, a);
    }
    if (step == DECODE_UP) DECODE(1 + (early ? down.n_tiles : shared_units) + candidates * up.n_tiles, (decode_up_kernel<UB, NT>), up, down, a, early);
    if (step == DECODE_DOWN) DECODE((early || !a.Ns ? 0 : down.n_tiles) + candidates * down.n_tiles, (decode_down_kernel<NT>), down, a, early);
#undef DECODE
    return hipGetLastError();
}
}  // namespace

hipError_t launch_decode(DecodeStep step, const GemmArgs& up, const GemmArgs& down, const DecodeArgs& a, bool nt, hipStream_t st) {
    // The shared experts run ahead, next to the top-k and to the routed gate/up GEMM, where the walk along their Ns * F of K (0.09 us
    // a sub-tile) hides behind the reads of that GEMM (4 H F bytes an expert at 5.8 TB/s): F cancels.  The experts that will be picked, at
    // least: one token's, three tenths of those that the batch can have.  Elsewhere the walk holds the launch up (layer, shared experts
    // ahead and not, us: 60 experts top-1 + 1 shared, H = 512, F = 12544, 1 token 64 and 45; 21 top-2 + 1, H = 576, F = 14720, 3
    // tokens 92 and 75; 19 top-2 + 2, H = 960, F = 7552, 1 token 69 and 58).
    const int candidates = a.pairs < a.E ? a.pairs : a.E;
    const float picked = fmaxf((float)a.k, 0.3f * candidates);
    const bool early = a.partial && a.Ns > 0 && picked * up.K >= 4078.f * a.Ns;
    const int units = (candidates + (early ? 0 : a.Ns)) * (up.N / 32);
    if (!nt) return launch_decode_units<2, false>(step, up, down, a, early, st);
    return up.K < 24 * 32 || (units > 1200 && units <= 2048) ? launch_decode_units<2, true>(step, up, down, a, early, st)
                                                             : launch_decode_units<1, true>(step, up, down, a, early, st);
}

hipError_t launch_decode_wide(DecodeStep step, const GemmArgs& up, const GemmArgs& down, const DecodeArgs& a, int col_blocks, bool nt, hipStream_t st) {
    const int candidates = a.pairs < a.E ? a.pairs : a.E, parts = (up.T + SMALL_ROWS - 1) / SMALL_ROWS;
    const int groups_up = a.Ns + candidates, groups_down = (a.Ns > 0) + candidates;
    const dim3 grid_up((unsigned)(1 + groups_up * parts * up.n_tiles)), grid_down((unsigned)(groups_down * parts * down.n_tiles)), block(64);
#define WIDE(grid_, K_, args_, groups_) hipLaunchKernelGGL((K_), grid_, block, 0, st, args_, a, parts, groups_)
    if (step == DECODE_UP) {
        if (nt) WIDE(grid_up, decode_wide_up_kernel<true>, up, groups_up);
        else WIDE(grid_up, decode_wide_up_kernel<false>, up, groups_up);
    } else if (step == DECODE_DOWN) {
        if (col_blocks == 2 && nt) WIDE(grid_down, (decode_wide_down_kernel<2, true>), down, groups_down);
        else if (col_blocks == 2) WIDE(grid_down, (decode_wide_down_kernel<2, false>), down, groups_down);
        else if (nt) WIDE(grid_down, (decode_wide_down_kernel<1, true>), down, groups_down);
        else WIDE(grid_down, (decode_wide_down_kernel<1, false>), down, groups_down);
    }
#undef WIDE
    return hipGetLastError();
}

}  // namespace moe
