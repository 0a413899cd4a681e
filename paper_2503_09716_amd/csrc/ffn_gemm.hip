// Grouped SwiGLU FFN as two grouped bf16 MFMA GEMMs with fp32 accumulation.
// (Sec. 2: each token is processed by its k selected experts; Sec. 4.2: experts see one large
// accumulated batch, so each expert's rows form a tall matrix and the GEMMs are compute bound.)
//
//   GEMM 1 (gated):  h[r, f]  = silu(X_e[r,:] . W1p_e[f,:]) * (X_e[r,:] . W3p_e[f,:])      -> bf16
//   GEMM 2        :  y[r, n]  = h[r,:] . W2p_e[n,:]                                        -> fp32 / bf16
// One tile routine serves both.  Weights and h are stored TILED: a matrix [N, K] is cut into
// blocks of 16 rows x 32 k (1 KiB) laid out block-row-major ([N/16][K/32] blocks), and the 64
// 16-byte pieces inside a block are in exactly the order the tile routine wants them in LDS
// (row-major rows of 64 bytes, piece slot = piece ^ ((row/4)&3)).  One direct-to-LDS load of a
// wavefront then reads 1 KiB of consecutive memory (8 full 128-byte lines) instead of 16
// half-lines from 16 distant rows, which halves the number of L1->L2 requests in flight; the
// L1's pending-request capacity, not bandwidth, is what the row-major form ran into
// (TCP_PENDING_STALL_CYCLES at half of all cycles).  x is read row-major through the gather
// unless a tiled copy exists.
//
// Tile routine (one workgroup = NW wavefronts in a WM x WN grid):
//   * macro tile: BM rows of X (32, 64, ... 384) x 256 rows of W (router: its experts; GEMM 1: 128 gate + 128
//     up rows, so the SiLU-gate product is formed in registers); K advances in sub-tiles of 32.
//     The tiles above 256 rows (4 waves side by side only) keep the accumulators of their last X blocks in VGPRs, the
//     256 AGPRs being full: fewer bytes from L2 per FLOP, and other numbers of rounds to choose from (plan.h).
//   * global -> LDS with buffer_load_dwordx4 ... lds (no VGPR round trip) into a ring of NS = 4
//     LDS stages (4 x 32 KiB at BM = 256, all 160 KiB at 384): the loads of sub-tile t+3 are issued while sub-tile t
//     is multiplied, so HBM latency has three sub-tiles of MFMA work to hide behind, and they
//     are spread between the MFMAs (one every few) instead of bursting after the barrier.
//     One barrier per sub-tile; s_waitcnt vmcnt(n) waits only for the sub-tile needed next.
//   * LDS layout: 64-byte rows (32 bf16), the four 16-byte pieces of a row XOR-swizzled by
//     (4 - row / 4) & 3 so that each of the four 16-lane passes in which the LDS serves a
//     16-byte MFMA operand read falls in distinct banks (block_swizzle).  The swizzle is applied by choosing which global piece each lane of the
//     direct-to-LDS load fetches, since the LDS side of that load is fixed (lane * 16 bytes).
//   * v_mfma_f32_16x16x32_bf16: one instruction multiplies a 16-row block of each operand over
//     the whole sub-tile.  In a register-only loop on this workload's data it sustains 1.98
//     PFLOP/s under the chip's power limit against 1.72 for v_mfma_f32_32x32x16_bf16 (both reach
//     2.47 on zeros): a quarter of the accumulator traffic per multiply-add.  GEMM 1 feeds W as
//     the row operand (a lane then owns 4 consecutive output columns of one row: 16-byte stores
//     of bf16 h after a swap between lanes), GEMM 2 feeds X as the row operand (a lane owns one output column: a store
//     instruction writes 4 rows x 64 contiguous bytes of fp32 y).
//   * each operand fragment has one register copy; it is refilled from the next LDS stage
//     right after its last use, so reads run ahead of the MFMAs that need them.  Up to 320 rows all X fragments
//     of a sub-tile are live; above, two chunks of them (a quarter of the rows each), which are walked with both halves of
//     W one after the other (more or smaller chunks, and chunks in lower tiles: the same or slower).  The
//     instruction stream is laid out by hand in small groups {MFMAs of one X block,
//     one or two LDS reads, at most one global load} fenced by scheduling barriers, so the
//     matrix pipe always has independent work queued.
//   * ragged tails: rows past the end of a group are clamped on load and masked on store;
//     a tile runs the lowest variant that holds its rows, so padded MFMA work stays small.
//
// Work distribution: a device-built list of m-tiles (plan.h) x n-tiles; workgroup ids are
// remapped so each XCD (ids are dealt round-robin over the 8 XCDs) receives runs of 32
// consecutive tiles (8 in short launches next to shared experts), and consecutive tiles sweep
// `group_m` m-tiles before moving along n, so the tiles resident on one XCD share weight panels
// and X panels in its L2.
#include <type_traits>
#include <utility>

#include "common.h"
#include "plan.h"

namespace moe {
namespace {

constexpr int BK = 32;              // K elements per LDS stage
constexpr int ROWB = BK * 2;        // bytes per LDS row
constexpr int WROWS = 256;          // W rows per macro tile
constexpr int NS = 4;               // LDS ring depth (deeper rings for the low tiles, up to 8 stages, measured the same)
constexpr int MAX_ROWS = PLAN_MAX_ROWS;   // tallest macro tile
constexpr int MAX_STAGE = (MAX_ROWS + WROWS) * ROWB;     // 40 KiB
constexpr int MAX_LDS = NS * MAX_STAGE;
constexpr int COMBINE_LDS = 2 * 64 * (256 * 4 + 16) + 256 * 64;   // epilogue of launch_down_combine
static_assert(COMBINE_LDS <= MAX_LDS, "LDS");

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef __attribute__((address_space(3))) char* lds_t;

// Buffer descriptor over [ptr, ptr + 4 GiB - 1) for raw (untyped) accesses.  The pointer is
// wave-uniform by construction; readfirstlane tells the compiler so (otherwise every load is
// wrapped in a waterfall loop).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* ptr) {
    const uint64_t v = (uint64_t)ptr;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, 0xFFFFFFFF, 0x00020000);
}

// 64 lanes x 16 bytes from (descriptor base + voff + soff) to LDS at l + lane*16 (l wave-uniform).
// The 16-byte form exists on gfx950 only; the host pass of hipcc must not see it.
template <int AUX = 0>
__device__ __forceinline__ void buffer_load16_to_lds(__amdgpu_buffer_rsrc_t rsrc, lptr_t l, uint32_t voff, int soff) {
#if defined(__gfx950__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, l, 16, voff, soff, 0, AUX);
#endif
}

// Descriptor over exactly [ptr, ptr + bytes): accesses at offsets >= bytes are dropped by hardware.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* ptr, uint32_t bytes) {
    const uint64_t v = (uint64_t)ptr;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ __forceinline__ void buffer_store_b32(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, float v) {
#if defined(__gfx950__)
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, voff, 0, 0);
#endif
}

__device__ __forceinline__ void buffer_store_bf16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, float v) {
#if defined(__gfx950__)
    const __bf16 b = (__bf16)v;
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, b), rsrc, voff, 0, 0);
#endif
}

__device__ __forceinline__ u32x4 buffer_load_b128(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff) {
#if defined(__gfx950__)
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, 0, 0);
#else
    return u32x4{};
#endif
}

__device__ __forceinline__ void buffer_store_b128(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, u32x4 v) {
#if defined(__gfx950__)
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, voff, 0, 0);
#endif
}

// Lanes 16..31 and 48..63 of a and lanes 0..15 and 32..47 of b change places; both halves as one piece.
__device__ __forceinline__ u32x4 swap_rows16(const u32x2 a, const u32x2 b) {
    u32x4 o = {0u, 0u, 0u, 0u};
#if defined(__gfx950__)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(a[i], b[i], false, false));
        o[i] = r[0];
        o[2 + i] = r[1];
    }
#endif
    return o;
}

// c += a (16 x 32, row operand) * b (32 x 16, column operand).  Written as inline assembly with
// the accumulator tied to an AGPR quad: left to itself the register allocator (all 256 AGPRs
// hold accumulators) routes part of them through temporaries, two to four copies per MFMA.
// Hazards the compiler would otherwise cover: the operands come from LDS reads it still
// tracks (s_waitcnt); an accumulator is re-used only a full sub-tile (>= 4 MFMAs, 64 cycles) later; the
// epilogue waits mfma_drain() before it reads accumulators.
__device__ __forceinline__ void mfma_16x16x32(f32x4& c, const bf16x8& a, const bf16x8& b) {
#if defined(__gfx950__)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
#endif
}
// The same with the accumulator in VGPRs: the X blocks of a tall tile that the 256 AGPRs do not hold.
__device__ __forceinline__ void mfma_16x16x32_v(f32x4& c, const bf16x8& a, const bf16x8& b) {
#if defined(__gfx950__)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
#endif
}
__device__ __forceinline__ void mfma_drain() {
#if defined(__gfx950__)
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#endif
}

// Hand-over point of the LDS ring: wait until at most N of this wave's direct-to-LDS loads
// are still in flight (they retire in order, so everything older has landed) and until this
// wave's own LDS reads have returned, then meet the other waves.  A bare s_barrier is used
// instead of __syncthreads(), whose release fence would drain ALL outstanding loads and so
// serialise the ring; the empty asm statements keep the compiler from moving LDS accesses
// across the barrier.
template <int N>
__device__ __forceinline__ void ring_sync() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0070);  // vmcnt(N) lgkmcnt(0), gfx9 encoding
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// NW wavefronts as a WM x (NW/WM) grid; TI = 32-row X blocks per wave; GATED = GEMM 1.
// ONCE: no other tile reads this one's W panel, so its loads are non-temporal (they do not displace what
// other tiles share): 8x7B, 32 rows per expert gate/up 335 -> 319 us, down 184 -> 168, 100 rows 377 -> 365, 203 -> 193;
// 160 experts, 2000 tokens gate/up 1105 -> 1050.  Where two tiles share a panel it costs as much (eight experts of
// 250 rows, down 266 -> 287), and above 128 rows it gains 1-3 %, less than a second copy of the variants costs.
// WR: rows of W per macro tile.  COMB, OF32: the layer's combine in the epilogue (launch_down_combine), of COMB rows a token.
template <int NW, int WM, int TI, bool GATED, bool UNIFORM = false, bool ONCE = false, int WR = WROWS, int COMB = 0, bool OF32 = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs& p, const TileDesc d, const int n_tile, char* lds, const CombineArgs* comb = nullptr) {
    constexpr int WN = NW / WM;
    constexpr int TJ = WR / 32 / WN;         // 32-row W blocks per wave
    constexpr int BM = WM * TI * 32;
    constexpr int NLX = (BM / 16 + NW - 1) / NW;   // X wave-loads (16 rows x 64 B) per wave per stage
    constexpr int NQX = NLX * NW;                  // X wave-loads per stage (region padded to a multiple of NW)
    constexpr int XBYTES = NQX * 1024;
    constexpr int NL = NLX + (WR / 16) / NW;    // all wave-loads per wave per stage
    constexpr int RING_STRIDE = NL * NW * 1024;    // bytes per ring stage
    static_assert(NS * RING_STRIDE <= MAX_LDS, "ring does not fit");
    constexpr int BN = GATED ? 128 : WR;    // output columns per macro tile
    constexpr int W_AUX = ONCE ? 2 : 0;      // cache policy of the W loads: 2 = non-temporal
    constexpr int TJH = TJ / 2;              // GATED: 32-row gate blocks per wave (= up blocks per wave)
    // The MFMA works on 16-row blocks (v_mfma_f32_16x16x32_bf16: one instruction spans a whole
    // K sub-tile of 32).  Per wave: XB blocks of X and WB blocks of W, the latter in two halves
    // of WBH (GEMM 1: gate blocks | up blocks).
    constexpr int XB = 2 * TI;
    constexpr int WB = 2 * TJ;
    constexpr int WBH = WB / 2;
    constexpr int XB_A = 64 / WB;            // X blocks whose accumulators fit the 256 AGPRs; the rest live in VGPRs
    // The X blocks are walked in NC chunks of CB, each chunk with both halves of W before the next.  XD fragments of X
    // are live: all of them (one chunk) up to 320 rows, two chunks above, where the accumulators leave no room for all.
    constexpr int NC = XB == 24 ? 4 : (XB == 22 ? 2 : 1);
    constexpr int CB = XB / NC;
    constexpr int XD = NC == 1 ? XB : 2 * CB;
    static_assert(NC * CB == XB && XB % XD == 0, "X blocks do not divide into chunks");
    // The hand-over of the ring comes before the first part (chunk, half of W) that reads the next stage.
    constexpr int SYNC_PART = NC == 1 ? 1 : 2 * NC - 3;
    constexpr int NL0 = SYNC_PART * CB * NL / (2 * XB);   // loads of an iteration issued before that
    static_assert(TJ >= 1 && (!GATED || TJ >= 2), "wave grid too wide");
    static_assert(BM <= MAX_ROWS, "tile too tall");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int K = p.K, N = p.N;
    const int n0 = n_tile * BN;
    const bool shared = d.srow >= 0;
    // K-split.  Router GEMM: srow = -1 - s, the operands of piece s start s*K further along and
    // its partial output goes to rows s*split_rows + ...  Down GEMM with tail_splits > 1: a short
    // tail is cut into tail_splits pieces along K; srow = -2 - u, u counting the pieces of all
    // split tails; piece u covers K range (u % tail_splits) * K/tail_splits .. and writes fp32
    // partials to rows u * SPLIT_TAIL_ROWS of out_partial.
    const bool tail_split = !GATED && p.tail_splits > 1 && d.srow <= -2;
    const int piece = tail_split ? -2 - d.srow : (shared ? 0 : -1 - d.srow);
    const int split = tail_split ? piece % p.tail_splits : piece;
    const int nseg = (!GATED && shared) ? p.nseg_shared : 1;
    const int KT = (tail_split ? K / p.tail_splits : K) / BK;   // sub-tiles per segment (>= 2)
    // K step in bytes: one 1 KiB block for tiled operands, 64 bytes along a row for row-major x
    constexpr int kstep_w = 1024;
    // A operand layout (bit 0: routed tiles, bit 1: shared tiles): h is tiled; x is row-major
    // (read through the gather, by shared experts and by the router) unless a tiled x_perm exists
    const bool a_tiled = ((shared ? p.a_tiled >> 1 : p.a_tiled) & 1) != 0;
    const int kstep_x = a_tiled ? 1024 : ROWB;
    const char* const a_base = shared ? p.a_shared : p.a_routed;
    const size_t a_seg_stride = (size_t)p.t_pad * (size_t)K * 2;   // one shared expert's block of h

    // ------------------------------------------------------------------ loader setup
    // Wave-load q fills LDS bytes [q*1024, q*1024+1024) of a stage: 16 rows x 4 pieces.
    // Lane l supplies row q*16 + l/4, slot l%4, which must hold logical piece (l%4) ^ block_swizzle(l/4).
    // This wave owns q = i*NW + wave; the X region is padded to a multiple of NW wave-loads so
    // that load i is an X load for i < NLX and a W load otherwise, for every wave.
    // Loads are buffer loads: address = operand base (SGPR descriptor) + per-lane offset (VGPR,
    // fixed for the whole tile) + K offset (SGPR, advanced per sub-tile), so the K loop needs no
    // vector address arithmetic at all.
    const int lrow = lane >> 2;
    const int lpiece = (lane & 3) ^ block_swizzle(lrow);
    uint32_t loff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int q = i * NW + wave;
        if (i < NLX) {
            int r = q * 16 + lrow;
            if (r > d.nrows - 1) r = d.nrows - 1;     // padded rows re-read the last valid row
            int grow = d.row0 + r;
            if (!a_tiled) {
                // x: row-major [rows, K]
                if (!shared && p.row_token) grow = p.row_token[grow];
                loff[i] = (uint32_t)grow * (uint32_t)p.lda_bytes + (uint32_t)(lpiece * 16);
            } else {
                // h: tiled; the piece this lane needs sits at slot piece ^ block_swizzle(row%16) of its row
                const int rr = grow & 15;
                loff[i] = (uint32_t)(grow >> 4) * (uint32_t)(p.kt_a * 1024) + (uint32_t)(rr * 64 + ((lpiece ^ block_swizzle(rr)) << 4));
            }
        } else {
            // W: tiled by the pack step, so LDS rows (q-NQX)*16 .. +15 of the W region
            // are one 1 KiB block: group index n0/16 + (q-NQX), in lane order.
            const int qw = q - NQX;
            int grp = (n0 >> 4) + (GATED ? (qw & 7) : qw);
            if (grp > (N >> 4) - 1) grp = (N >> 4) - 1;
            loff[i] = (uint32_t)grp * (uint32_t)(p.kt_w * 1024) + (uint32_t)(lane * 16);
        }
    }
    lds_t const ring = (lds_t)lds;
    __amdgpu_buffer_rsrc_t rs_x, rs_w, rs_u;   // X, W (gate / down), W (up)
    int koff_x = 0, koff_w = 0;                // byte offsets along K of the sub-tile being loaded

    // Enqueues direct-to-LDS load i of the sub-tile at `koff` into ring stage `stage`.
    auto issue_one = [&](const int i, const int stage) __attribute__((always_inline)) {
        lptr_t dst = (lptr_t)(ring + stage * RING_STRIDE + (i * NW + wave) * 1024);
        if (i < NLX) buffer_load16_to_lds(rs_x, dst, loff[i], koff_x);
        else if (GATED && (i - NLX) * NW >= 8) buffer_load16_to_lds<W_AUX>(rs_u, dst, loff[i], koff_w);
        else buffer_load16_to_lds<W_AUX>(rs_w, dst, loff[i], koff_w);
    };

    // ------------------------------------------------------------------ reader setup
    // Lane l reads row (l & 15) of a 16-row block, logical piece l >> 4 (k = 8*(l>>4) .. +7),
    // stored at slot piece ^ block_swizzle(row).  Block bases are multiples of 16 rows, so the
    // swizzle term depends on the lane only.
    const int rl = lane & 15, g = lane >> 4;
    const int bx0 = wm * TI;                       // in 32-row units
    const int bw0 = GATED ? wn * TJH : wn * TJ;    // in 32-row units
    const uint32_t offL = (uint32_t)(rl * ROWB + ((g ^ block_swizzle(rl)) << 4));
    const uint32_t offX = offL + (uint32_t)(bx0 * 32 * ROWB);
    const uint32_t offW = offL + (uint32_t)(XBYTES + bw0 * 32 * ROWB);

    // COMB (k of the combine, 0 = none): this thread's token's rows of y_perm and weights, asked for here and used in the epilogue
    uint32_t pick[COMB > 0 ? COMB : 1];
    float weight[COMB > 0 ? COMB : 1];
    if constexpr (COMB > 0) {
        const size_t t = (size_t)(d.row0 + min((int)threadIdx.x, d.nrows - 1)) * COMB;
#pragma unroll
        for (int j = 0; j < COMB; ++j) {
            pick[j] = (uint32_t)comb->inv_perm[t + j];
            weight[j] = comb->w[t + j];
        }
    }

    f32x4 acc[WB][XB];
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
        for (int i = 0; i < XB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;

    // Operand fragments: XD X blocks, and the W blocks of one sub-tile in two halves.  wA is used by the first half of
    // every chunk and refilled (from the NEXT stage) during the second half of the last; wB by the second
    // halves, refilled during the first half of the first chunk; an X fragment is refilled with the block XD
    // further on (past the last one: of the next stage) right after its last MFMA.  So no fragment needs a second copy.
    bf16x8 xf[XD], wA[WBH], wB[WBH];
    typedef __attribute__((address_space(3))) const bf16x8* frag_ptr_t;
    auto read_x = [&](const int stage, const int i) __attribute__((always_inline)) {
        xf[i % XD] = *(frag_ptr_t)(ring + stage * RING_STRIDE + offX + i * 16 * ROWB);
    };
    // W block jj of half hf: GEMM 2: rows (hf*WBH + jj)*16; GEMM 1: gate rows jj*16 | up rows 128 + jj*16
    auto read_w = [&](const int stage, const int hf, const int jj) __attribute__((always_inline)) {
        const int rows = GATED ? hf * 128 + jj * 16 : (hf * WBH + jj) * 16;
        const bf16x8 v = *(frag_ptr_t)(ring + stage * RING_STRIDE + offW + rows * ROWB);
        if (hf == 0) wA[jj] = v;
        else wB[jj] = v;
    };

    // Part P of a sub-tile: chunk P / 2 with half HF = P % 2 of the W blocks, CB groups of WBH MFMAs with one X block.
    // Second halves refill X fragments, from stage `cur` or, where RD, from stage `nxt`; W as above.
    // The direct-to-LDS loads of an iteration are spread over its 2 * XB groups (LD).
    auto part = [&](auto p_tag, auto rd_tag, auto ld_tag, const int cur, const int nxt, const int ld_stage) __attribute__((always_inline)) {
        constexpr int P = decltype(p_tag)::value, C = P / 2, HF = P % 2;
        constexpr bool RD = decltype(rd_tag)::value;
        constexpr bool LD = decltype(ld_tag)::value;
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            const int i = C * CB + u;
#pragma unroll
            for (int jj = 0; jj < WBH; ++jj) {
                const int j = HF * WBH + jj;
                const bf16x8 w = HF == 0 ? wA[jj] : wB[jj];
                if (i < XB_A) {
                    if (GATED || COMB) mfma_16x16x32(acc[j][i], w, xf[i % XD]);
                    else mfma_16x16x32(acc[j][i], xf[i % XD], w);
                } else {
                    if (GATED || COMB) mfma_16x16x32_v(acc[j][i], w, xf[i % XD]);
                    else mfma_16x16x32_v(acc[j][i], xf[i % XD], w);
                }
            }
            if (HF == 1) {
                if (i + XD < XB) read_x(cur, i + XD);
                else if (RD) read_x(nxt, i + XD - XB);
            }
            // the WBH W reads of a half go out with the first groups
            constexpr int RPGW = (WBH + CB - 1) / CB;
            if (P == 0 || (P == 2 * NC - 1 && RD)) {
#pragma unroll
                for (int jj = u * RPGW; jj < (u + 1) * RPGW && jj < WBH; ++jj) read_w(P == 0 ? cur : nxt, P == 0 ? 1 : 0, jj);
            }
            if (LD) {
                constexpr int G = 2 * XB;
                const int q = P * CB + u;
#pragma unroll
                for (int l = (q * NL) / G; l < ((q + 1) * NL) / G; ++l) issue_one(l, ld_stage);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // One sub-tile: its parts in order, `sync` before part SYNC_PART.
    auto sub_tile = [&](auto rd_tag, auto ld_tag, const int cur, const int nxt, const int ld_stage, auto sync) __attribute__((always_inline)) {
        auto run = [&](auto p_tag) __attribute__((always_inline)) {
            if (decltype(p_tag)::value == SYNC_PART) sync();
            part(p_tag, rd_tag, ld_tag, cur, nxt, ld_stage);
        };
        [&]<int... P>(std::integer_sequence<int, P...>) __attribute__((always_inline)) {
            (run(std::integral_constant<int, P>{}), ...);
        }(std::make_integer_sequence<int, 2 * NC>{});
    };
    using T_ = std::true_type;
    using F_ = std::false_type;

    // GEMM 2 on shared experts walks `nseg` K-concatenated segments (one per shared expert);
    // every other tile has one segment.  The pipeline drains and restarts between segments.
    for (int seg = 0; seg < nseg; ++seg) {
        // the descriptors span 4 GiB - 1; bounds are kept by the row clamps above
        // a K piece starts `split` pieces along: K*2 bytes per piece in a row-major row, KT blocks of
        // 1 KiB in a tiled operand (the packed W is always tiled)
        const size_t piece_shift = (size_t)split * (size_t)KT * 1024;
        rs_x = uniform_rsrc(a_base + (size_t)seg * a_seg_stride + (tail_split ? piece_shift : (size_t)split * (size_t)K * 2));
        // UNIFORM (router GEMM): one packed matrix, K-split s starts s * w_uniform_stride bytes along
        if (UNIFORM) rs_w = uniform_rsrc(p.w_uniform + (size_t)d.group * (size_t)p.w_uniform_stride);
        else rs_w = uniform_rsrc((const char*)p.w_a[d.group + seg] + (tail_split ? piece_shift : 0));
        if (GATED) rs_u = uniform_rsrc(p.w_b[d.group]);
        koff_x = 0;
        koff_w = 0;
        // prologue: sub-tiles 0 .. NS-2 go out, wait for sub-tile 0
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
            if (s < KT) {
#pragma unroll
                for (int i = 0; i < NL; ++i) issue_one(i, s);
                koff_x += kstep_x;
                koff_w += kstep_w;
            }
        }
        if (KT >= NS - 1) ring_sync<(NS - 2) * NL>();
        else ring_sync<0>();
        // Same order as the reads inside the loop (the first-half W blocks among the first X
        // blocks): LDS reads return in order, and where the two paths into the loop meet the
        // compiler waits for whichever leaves fewer reads outstanding behind the registers the
        // first MFMAs need.  With the W blocks read last here (where the scheduler puts them if
        // left alone), that was a wait for every read of the previous iteration at the top of
        // each sub-tile.
        constexpr int RPGW0 = (WBH + XD - 1) / XD;
#pragma unroll
        for (int i = 0; i < XD; ++i) {
            read_x(0, i);
#pragma unroll
            for (int jj = i * RPGW0; jj < (i + 1) * RPGW0 && jj < WBH; ++jj) read_w(0, 0, jj);
            __builtin_amdgcn_sched_barrier(0);   // keeps the compiler from moving the W reads to the end
        }

        int t = 0;
        // steady state: sub-tile t is multiplied, sub-tile t+NS-1 is loaded
        for (; t + NS - 1 < KT; ++t) {
            // Sub-tile t+1 has landed once only the younger loads are outstanding.  The same
            // barrier frees stage t % NS for the loads of the NEXT iteration: its last reads were
            // issued before and have returned (lgkmcnt(0)) before any wave passes.
            sub_tile(T_{}, T_{}, t % NS, (t + 1) % NS, (t + NS - 1) % NS,
                     [] __attribute__((always_inline)) { ring_sync<(NS - 3) * NL + NL0>(); });
            koff_x += kstep_x;
            koff_w += kstep_w;
        }
        // tail: nothing left to load; conservative waits
        auto drain = [] __attribute__((always_inline)) { ring_sync<0>(); };
        for (; t < KT - 1; ++t) sub_tile(T_{}, F_{}, t % NS, (t + 1) % NS, 0, drain);
        sub_tile(F_{}, F_{}, t % NS, 0, 0, drain);   // its barrier: every wave is done reading the ring before the next segment refills it
    }

    // ------------------------------------------------------------------ epilogue
    // Accumulator block (j, i) is 16 x 16; a lane holds 4 registers: the block's MFMA-row-operand
    // index 4*(lane/16) + r and column-operand index lane%16.
    mfma_drain();
    if constexpr (COMB > 0) {
        static_assert(!GATED && NW == 4 && WM == 1 && BM <= 256 && COMB <= 8, "one row to a thread");
        // The layer's last step: out[t] = sum_j w[t, j] * y_perm[inv_perm[t, j]] + this GEMM's row t, in combine_kernel's order.
        // 64 rows of the tile at a time go through LDS, so that a wave reads 512 consecutive bytes of a row of y_perm: with
        // the accumulators' own columns, 64 bytes of 16 rows to a load, the loads took twice as long (every row is
        // another page).  W is the row operand as in GEMM 1 (a lane has 4 consecutive columns of a row).  The ring is free: every wave is
        // past the last barrier.  LDS: two buffers of 64 rows, then the tokens' row offsets and weights.
        typedef __attribute__((address_space(3))) u32x4* lds4_t;
        constexpr int ROW = 256 * 4 + 16, BUF = 64 * ROW, META = 2 * BUF;
        static_assert(META + BM * 64 <= COMBINE_LDS, "LDS");
        const uint32_t rowbytes = (uint32_t)N * 2u;
        if ((int)threadIdx.x < BM) {
            u32x4 v[4] = {};
#pragma unroll
            for (int j = 0; j < COMB; ++j) {
                v[j >> 2][j & 3] = pick[j] * rowbytes;
                v[2 + (j >> 2)][j & 3] = __float_as_uint(weight[j]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((q & 1) * 4 < COMB) *((lds4_t)(ring + META + threadIdx.x * 64) + q) = v[q];
        }
        ring_sync<63>();   // LDS only: nothing here waits for loads
        constexpr uint32_t esz = OF32 ? 4 : 2;
        constexpr int CHUNKS = BM / 64, STEPS = CHUNKS * 8, DEPTH = 3;   // a step: two rows of the wave's 16 (4 and 5 steps on their way: no change)
        const __amdgpu_buffer_rsrc_t rs_y = uniform_rsrc(comb->y_perm);
        const __amdgpu_buffer_rsrc_t rs_o = tile_rsrc(comb->out + (size_t)d.row0 * (size_t)N * esz, (uint32_t)d.nrows * (uint32_t)N * esz);
        const int cols = (lane & 31) * 8, col = n0 + cols;
        const bool col_ok = col < N;
        const uint32_t ycol = (uint32_t)min(col, N - 8) * 2u;
        auto row_of = [&](const int st) __attribute__((always_inline)) { return (st >> 3) * 64 + wave * 16 + (st & 7) * 2 + (lane >> 5); };
        u32x4 y[DEPTH][COMB];
        auto gather = [&](const int st) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q * 4 < COMB; ++q) {
                const u32x4 at = *((lds4_t)(ring + META + row_of(st) * 64) + q);
#pragma unroll
                for (int j = q * 4; j < COMB && j < q * 4 + 4; ++j) y[st % DEPTH][j] = buffer_load_b128(rs_y, at[j & 3] + ycol);
            }
        };
#pragma unroll
        for (int st = 0; st < DEPTH - 1; ++st) gather(st);
#pragma unroll
        for (int ch = 0; ch < CHUNKS; ++ch) {
            const lds_t buf = ring + (ch & 1) * BUF;
#pragma unroll
            for (int i = 4 * ch; i < 4 * ch + 4; ++i)
#pragma unroll
                for (int j = 0; j < WB; ++j) {
                    u32x4 v;   // read here, not earlier (as in store_tile below)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        uint32_t a;
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a) : "a"(acc[j][i][q]) : "memory");
                        v[q] = a;
                    }
                    *(lds4_t)(buf + ((i & 3) * 16 + rl) * ROW + (bw0 * 32 + j * 16 + g * 4) * 4) = v;
                }
            // one barrier to a buffer: the next write into it comes after the barrier of the other one, and so after every wave's reads
            ring_sync<63>();
#pragma unroll
            for (int st = ch * 8; st < ch * 8 + 8; ++st) {
                if (st + DEPTH - 1 < STEPS) gather(st + DEPTH - 1);
                __builtin_amdgcn_sched_barrier(0);
                const int row = row_of(st);
                float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q * 4 < COMB; ++q) {
                    const u32x4 w = *((lds4_t)(ring + META + row * 64) + 2 + q);
#pragma unroll
                    for (int j = q * 4; j < COMB && j < q * 4 + 4; ++j)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint32_t v = y[st % DEPTH][j][e >> 1];
                            sum[e] = fmaf(__uint_as_float(w[j & 3]), __uint_as_float(e & 1 ? v & 0xffff0000u : v << 16), sum[e]);
                        }
                }
                const lds4_t own = (lds4_t)(buf + (row & 63) * ROW + cols * 4);
                const u32x4 lo = own[0], hi = own[1];
#pragma unroll
                for (int e = 0; e < 4; ++e) { sum[e] += __uint_as_float(lo[e]); sum[4 + e] += __uint_as_float(hi[e]); }
                // offsets of rows past the end (up to 127 * N * 4) may wrap, so the descriptor cannot be left to drop them
                const bool ok = col_ok && row < d.nrows;
                const uint32_t at = ok ? ((uint32_t)row * (uint32_t)N + (uint32_t)col) * esz : 0xFFFFFFF0u;
                if (OF32) {
                    buffer_store_b128(rs_o, at, u32x4{__float_as_uint(sum[0]), __float_as_uint(sum[1]), __float_as_uint(sum[2]), __float_as_uint(sum[3])});
                    buffer_store_b128(rs_o, ok ? at + 16 : at, u32x4{__float_as_uint(sum[4]), __float_as_uint(sum[5]), __float_as_uint(sum[6]), __float_as_uint(sum[7])});
                } else {
                    bf16x8 o;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)sum[e];
                    buffer_store_b128(rs_o, at, __builtin_bit_cast(u32x4, o));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return;
    }
    char* out = shared ? p.out_shared : (tail_split ? p.out_partial : p.out_routed);
    const int orow_base = tail_split ? piece * SPLIT_TAIL_ROWS
                                     : (shared ? (GATED ? d.srow : 0) : split * p.split_rows) + d.row0;
    if (GATED) {
        // W is the row operand: the lane owns output row (X row) lane%16 of block i and the 4
        // consecutive columns 4*(lane/16) .. +3 of gate block j; the up value of the same
        // element sits in the same lane and register of block WBH + j.  Gate blocks j and j + 1 are the two halves
        // of one 32-column block of h (row%16 at 64 bytes each, piece slot = piece ^ block_swizzle(row%16)).  Lanes 16 apart
        // swap halves, so that each has one 16-byte piece and a store instruction covers 16 rows x 64 contiguous bytes.
        // VALU-bound (a quarter-rate exponential and reciprocal per element), so: no branch between the elements, whose
        // chains then overlap, and no address arithmetic (row block i is i * hstep bytes on, rows past the group's end
        // get an offset that the descriptor drops).  Gate/up GEMM against 8-byte pieces behind a branch each: 64 experts, 16384 tokens
        // 1148 -> 1135 us, 160 experts, 32768 tokens 6029 -> 5972, 8x7B, 4096 tokens 1365 -> 1352.
        const int orow = orow_base + bx0 * 32, rr = (orow + rl) & 15;
        const uint32_t hstep = (uint32_t)(N >> 5) * 1024u;   // bytes of 16 rows of h
        const uint32_t hblocks = (uint32_t)(((orow_base & 15) + d.nrows + 15) >> 4);
        const __amdgpu_buffer_rsrc_t rs_h = tile_rsrc(out + (size_t)(orow_base >> 4) * hstep, hblocks * hstep);
        const uint32_t hoff = (uint32_t)(((orow + rl) >> 4) - (orow_base >> 4)) * hstep +
                              (uint32_t)(rr * 64 + ((((g >> 1) + 2 * (g & 1)) ^ block_swizzle(rr)) << 4));
#pragma unroll
        for (int j = 0; j < WBH; j += 2) {
            const int col = n0 + bw0 * 32 + j * 16;   // wave-uniform; N is a multiple of 64
            if (col >= N) break;
            const uint32_t at = hoff + (uint32_t)(col >> 5) * 1024u;
#pragma unroll
            for (int i = 0; i < XB; ++i) {
                u32x2 o[2];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    bf16x4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float gv = acc[j + b][i][q], uv = acc[WBH + j + b][i][q];
                        // silu(g) * u with the hardware reciprocal (1 ulp): far below the bf16 rounding of h
                        v[q] = (__bf16)(gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv)) * uv);
                    }
                    o[b] = __builtin_bit_cast(u32x2, v);
                }
                const bool row_ok = bx0 * 32 + i * 16 + rl < d.nrows;
                buffer_store_b128(rs_h, row_ok ? at + (uint32_t)i * hstep : 0xFFFFFFFFu, swap_rows16(o[0], o[1]));
                if (i % 2) __builtin_amdgcn_sched_barrier(0);   // two block rows at a time: keeps accumulator reads from piling up
            }
        }
    } else {
        // GEMM 2 / router GEMM: X is the row operand, so the lane owns output column lane%16 of W
        // block j and the 4 consecutive rows 4*(lane/16) .. +3 of X block i.  One store
        // instruction writes 4 rows x 64 contiguous bytes (fp32).  Rows past the end of the
        // group and columns past N fall outside the buffer descriptor, which spans exactly the
        // valid rows of the 16-row block being stored, and are dropped by hardware.
        // The descriptor is rebuilt (scalar work) for every 16-row block of X so that the row
        // part of the address is in its base and the 16 per-lane offsets {W block j, row r} are
        // computed once per tile: a store then needs no vector address arithmetic and no
        // registers beyond its data.
        auto store_tile = [&](auto f32_tag) __attribute__((always_inline)) {
            constexpr bool F32 = decltype(f32_tag)::value;
            constexpr int esz = F32 ? 4 : 2;
            const uint32_t rowbytes = (uint32_t)N * (uint32_t)esz;
            uint32_t vcol[WB][4];
#pragma unroll
            for (int j = 0; j < WB; ++j) {
                const int col = n0 + bw0 * 32 + j * 16 + rl;
                const uint32_t base = col < N ? (uint32_t)(g * 4) * rowbytes + (uint32_t)col * esz : 0x80000000u;
#pragma unroll
                for (int r = 0; r < 4; ++r) vcol[j][r] = base + (uint32_t)r * rowbytes;
            }
#pragma unroll
            for (int i = 0; i < XB; ++i) {
                const int r0 = bx0 * 32 + i * 16;                          // wave-uniform
                const int left = min(max(d.nrows - r0, 0), 16);            // valid rows of this block
                const __amdgpu_buffer_rsrc_t rs_o =
                    tile_rsrc(out + (size_t)(orow_base + r0) * rowbytes, (uint32_t)left * rowbytes);
#pragma unroll
                for (int j = 0; j < WB; ++j) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (F32) {
                            buffer_store_b32(rs_o, vcol[j][r], acc[j][i][r]);
                        } else {
                            // read the accumulator here, not earlier: left alone the compiler copies all
                            // accumulators to VGPRs ahead of the first store and spills to make room
                            float v;
                            if (i < XB_A) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[j][i][r]) : "memory");
                            else asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "v"(acc[j][i][r]) : "memory");
                            buffer_store_bf16(rs_o, vcol[j][r], v);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);   // one block row at a time
            }
        };
        if (tail_split || ((shared ? p.out_fp32 >> 1 : p.out_fp32) & 1)) store_tile(T_{});
        else store_tile(F_{});
    }
}

// Workgroup id -> position in the tile order.  Hardware deals consecutive workgroup ids to the
// 8 XCDs in turn; inside each stretch of 8 * run ids, XCD x is given tiles [run * x, run * (x + 1)).
// Only whole rounds of 256 tiles are dealt in runs of 32, and whole stretches in shorter ones.
__device__ __forceinline__ int tile_order(const int wg, const int total, const int run) {
    if (!run) return wg;
    const int span = run * 8;   // 64 or 256
    if (wg >= (total & ~(span - 1))) return wg;
    const int r = wg & (span - 1);
    return (wg - r) + (r & 7) * run + (r >> 3);
}

// Tile picked by this workgroup (false: nothing to do).  The first n_run entries of the m-tile
// list are cut into runs of group_m consecutive m-tiles; the tiles of a run are visited
// m-fastest, then along n, so tiles that run at the same time share W panels (same n, same
// group) and X panels (same m) in L2.  (Runs of a fixed length that cross group boundaries
// measured 5-12 % faster than runs fitted to each group.)  Entries past n_run are tail tiles
// of different groups: they are walked along n, which shares the X panel.
__device__ __forceinline__ bool pick_tile(const GemmArgs& p, const bool gated, TileDesc& d, int& n_tile, bool& once, bool& full) {
    const int count = gated ? p.plan->n_gate_up : p.plan->n_down;
    const int n_run = gated ? p.plan->n_run_up : p.plan->n_run_down;
    // Only whole rounds of 256 REAL tiles are dealt to the XCDs in runs of 32, stretches of 64 in runs of 8 (the grid is an upper
    // bound of the tile count, and how far the runs reach must not depend on it); the last,
    // partial round keeps the hardware's own order, which spreads it over all eight XCDs.  In
    // runs it would sit on the first few XCDs and leave the L2s and fabric links of the others
    // idle: a launch of 128 tiles measured 251 us on four XCDs against 210 us on eight, the
    // second of two rounds 6 % more; over the Mixtral-shaped layer from 1024 to 8192 tokens the
    // gate/up GEMM is 0.7-2.6 % faster this way, the named workloads are unchanged.
    const int L = tile_order(blockIdx.x, count * p.n_tiles, gated ? p.plan->xcd_run_up : p.plan->xcd_run_down);
    const int run_positions = n_run * p.n_tiles;
    int mt;
    if (L < run_positions) {
        const int per_super = p.group_m * p.n_tiles;
        const int sr = L / per_super;
        const int rem = L - sr * per_super;
        const int mt0 = sr * p.group_m;
        const int gm = min(p.group_m, n_run - mt0);
        n_tile = rem / gm;
        mt = mt0 + (rem - n_tile * gm);
    } else {
        const int rem = L - run_positions;
        mt = n_run + rem / p.n_tiles;
        n_tile = rem - (mt - n_run) * p.n_tiles;
    }
    if (mt >= count) return false;  // uniform for the workgroup
    d = p.descs[mt];
    once = (d.nrows & TILE_ONCE) != 0;
    full = (d.nrows & TILE_FULL) != 0;
    d.nrows &= TILE_ROWS_MASK;
    return true;
}

// 4 wavefronts (one per SIMD, up to 512 registers each), wave grid WM x 4/WM.
template <int WM, bool GATED>
__global__ __launch_bounds__(256, 1) void ffn_gemm_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    TileDesc d;
    int n_tile;
    bool once, full;
    if (!pick_tile(p, GATED, d, n_tile, once, full)) return;
    // 32-row blocks that hold real rows; 9 or 10: a tall tile (the plan kernel makes them for this wave grid only)
    const int blocks = d.nrows > 256 ? (d.nrows + 31) >> 5 : (p.small_tiles && !full ? (d.nrows + 31) >> 5 : 8);
    if (WM == 2) {
        if (blocks > 4) gemm_tile<4, 2, 4, GATED>(p, d, n_tile, lds);
        else if (blocks > 2) gemm_tile<4, 2, 2, GATED>(p, d, n_tile, lds);
        else gemm_tile<4, 2, 1, GATED>(p, d, n_tile, lds);
    } else {
        if (blocks > 11) gemm_tile<4, 1, 12, GATED>(p, d, n_tile, lds);
        else if (blocks > 10) gemm_tile<4, 1, 11, GATED>(p, d, n_tile, lds);
        else if (blocks > 9) gemm_tile<4, 1, 10, GATED>(p, d, n_tile, lds);
        else if (blocks > 8) gemm_tile<4, 1, 9, GATED>(p, d, n_tile, lds);
        else if (blocks > 7) gemm_tile<4, 1, 8, GATED>(p, d, n_tile, lds);
        else if (blocks > 6) gemm_tile<4, 1, 7, GATED>(p, d, n_tile, lds);
        else if (blocks > 5) gemm_tile<4, 1, 6, GATED>(p, d, n_tile, lds);
        else if (blocks > 4) gemm_tile<4, 1, 5, GATED>(p, d, n_tile, lds);
        else if (once) {
            if (blocks > 3) gemm_tile<4, 1, 4, GATED, false, true>(p, d, n_tile, lds);
            else if (blocks > 2) gemm_tile<4, 1, 3, GATED, false, true>(p, d, n_tile, lds);
            else if (blocks > 1) gemm_tile<4, 1, 2, GATED, false, true>(p, d, n_tile, lds);
            else gemm_tile<4, 1, 1, GATED, false, true>(p, d, n_tile, lds);
        }
        else if (blocks > 3) gemm_tile<4, 1, 4, GATED>(p, d, n_tile, lds);
        else if (blocks > 2) gemm_tile<4, 1, 3, GATED>(p, d, n_tile, lds);
        else if (blocks > 1) gemm_tile<4, 1, 2, GATED>(p, d, n_tile, lds);
        else gemm_tile<4, 1, 1, GATED>(p, d, n_tile, lds);
    }
}

// Router GEMM: every K-split s covers all T rows in tiles of 64 * TI rows and 64 * TJ experts (all of them, or
// p.n_tiles tiles side by side); nothing to look up.  What a
// CU loads bounds it, so the tile has no more rows of the gate matrix than there are experts (in blocks of 64; all
// 256 rows of the FFN's tile before: 64 experts, 3001 tokens 17.2 -> 13.2 us, 16384 35.5 -> 28.6; 160 experts, 2000 tokens 29.9 -> 24.9).
template <int TI, int TJ>
__global__ __launch_bounds__(256, 2) void route_gemm_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int mt = blockIdx.x / p.n_tiles, n = blockIdx.x - mt * p.n_tiles, s = mt / p.uniform_per, m = mt - s * p.uniform_per;
    if (s >= p.uniform_splits) return;
    TileDesc d;
    d.group = s;
    d.row0 = m * 64 * TI;
    d.nrows = min(64 * TI, p.T - d.row0);
    d.srow = -1 - s;
    gemm_tile<4, 2, TI, false, true, false, 64 * TJ>(p, d, n, lds);
}

// The shared experts' down GEMM, all of them along K, with the combine behind it; tiles of 256 tokens by arithmetic, in the order of
// pick_tile.  Bound by the matrix cores, and in the epilogue by the latency of rows of y_perm from memory.  Against the
// tiles in the list, fp32 y_shared written and read, and combine_kernel: 160 experts top-6 + 2 shared, H = 5120, F = 1536, 32768 tokens, down
// and combine 3856 -> 3652 us; 64 experts, H = 2048, F = 1408, 16384 tokens 763 -> 716.
template <int K, bool OF32>
__global__ __launch_bounds__(256, 1) void ffn_down_combine_kernel(const GemmArgs p, const CombineArgs c) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int L = tile_order(blockIdx.x, p.uniform_per * p.n_tiles, 32);
    const int per_super = p.group_m * p.n_tiles, sr = L / per_super, rem = L - sr * per_super;
    const int mt0 = sr * p.group_m, gm = min(p.group_m, p.uniform_per - mt0);
    const int n_tile = rem / gm, mt = mt0 + (rem - n_tile * gm);
    TileDesc d;
    d.group = p.shared_group;
    d.row0 = mt * 256;
    d.nrows = min(256, p.T - d.row0);
    d.srow = 0;
    if (d.nrows > 128) gemm_tile<4, 1, 8, false, false, false, WROWS, K, OF32>(p, d, n_tile, lds, &c);
    else gemm_tile<4, 1, 4, false, false, false, WROWS, K, OF32>(p, d, n_tile, lds, &c);
}

// 8 wavefronts (two per SIMD, up to 256 registers each), wave grid WM x 8/WM: while one wave
// of a SIMD waits at the ring barrier or on LDS, the other keeps the matrix pipe fed.
template <int WM, bool GATED>
__global__ __launch_bounds__(512, 2) void ffn_gemm_kernel8(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    TileDesc d;
    int n_tile;
    bool once, full;
    if (!pick_tile(p, GATED, d, n_tile, once, full)) return;
    const int blocks = p.small_tiles ? (d.nrows + 31) >> 5 : 8;
    if (WM == 2) {
        if (blocks > 4) gemm_tile<8, 2, 4, GATED>(p, d, n_tile, lds);
        else if (blocks > 2) gemm_tile<8, 2, 2, GATED>(p, d, n_tile, lds);
        else gemm_tile<8, 2, 1, GATED>(p, d, n_tile, lds);
    } else {
        if (blocks > 4) gemm_tile<8, 4, 2, GATED>(p, d, n_tile, lds);
        else gemm_tile<8, 4, 1, GATED>(p, d, n_tile, lds);
    }
}

// The lists from expert_offsets in a launch of their own (staged calls, streamed passes, large batches; moe_layer
// otherwise builds them in the permutation's last launch).
__global__ __launch_bounds__(256) void ffn_plan_kernel(const PlanArgs p) { plan_list(p, blockIdx.x, p.offsets); }

// y_perm[row0 + r, :] of split tail q = sum over its K pieces of the fp32 partials, added in
// piece order (one thread per 4 columns, one workgroup per row): deterministic.
__global__ __launch_bounds__(256) void split_tail_reduce_kernel(const PlanHeader* __restrict__ plan,
                                                                const SplitTail* __restrict__ tails,
                                                                const float* __restrict__ partial, int splits, int H,
                                                                char* __restrict__ y, int y_fp32) {
    const int q = blockIdx.x / SPLIT_TAIL_ROWS, r = blockIdx.x % SPLIT_TAIL_ROWS;
    if (q >= plan->n_split_tails) return;
    const SplitTail t = tails[q];
    if (r >= t.nrows) return;
    for (int c = threadIdx.x * 4; c < H; c += 256 * 4) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int sp = 0; sp < splits; ++sp) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(partial + ((size_t)(q * splits + sp) * SPLIT_TAIL_ROWS + r) * H + c);
            acc += v;
        }
        const size_t at = (size_t)(t.row0 + r) * H + c;
        if (y_fp32) {
            *reinterpret_cast<f32x4*>(y + at * 4) = acc;
        } else {
            bf16x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (__bf16)acc[i];
            *reinterpret_cast<bf16x4*>(y + at * 2) = o;
        }
    }
}

}  // namespace

hipError_t launch_split_tail_reduce(const moe_shape& s, const PlanHeader* plan, const SplitTail* tails, const float* partial,
                                    int splits, void* y_perm, bool y_fp32, hipStream_t st) {
    hipLaunchKernelGGL(split_tail_reduce_kernel, dim3((unsigned)(s.E * SPLIT_TAIL_ROWS)), dim3(256), 0, st, plan, tails, partial,
                       splits, s.H, (char*)y_perm, y_fp32 ? 1 : 0);
    return hipGetLastError();
}

hipError_t ffn_gemm_init() {
    hipError_t e;
#define SET_LDS(K_)                                                                                            \
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&K_), hipFuncAttributeMaxDynamicSharedMemorySize,    \
                            MAX_LDS);                                                                          \
    if (e != hipSuccess) return e;
    SET_LDS((ffn_gemm_kernel<2, true>))
    SET_LDS((ffn_gemm_kernel<2, false>))
    SET_LDS((route_gemm_kernel<1, 1>))
    SET_LDS((route_gemm_kernel<1, 2>))
    SET_LDS((route_gemm_kernel<1, 3>))
    SET_LDS((route_gemm_kernel<1, 4>))
    SET_LDS((route_gemm_kernel<2, 1>))
    SET_LDS((route_gemm_kernel<2, 2>))
    SET_LDS((route_gemm_kernel<2, 3>))
    SET_LDS((route_gemm_kernel<2, 4>))
    SET_LDS((ffn_gemm_kernel<1, true>))
    SET_LDS((ffn_gemm_kernel<1, false>))
    SET_LDS((ffn_down_combine_kernel<4, false>))
    SET_LDS((ffn_down_combine_kernel<4, true>))
    SET_LDS((ffn_down_combine_kernel<5, false>))
    SET_LDS((ffn_down_combine_kernel<5, true>))
    SET_LDS((ffn_down_combine_kernel<6, false>))
    SET_LDS((ffn_down_combine_kernel<6, true>))
    SET_LDS((ffn_down_combine_kernel<7, false>))
    SET_LDS((ffn_down_combine_kernel<7, true>))
    SET_LDS((ffn_down_combine_kernel<8, false>))
    SET_LDS((ffn_down_combine_kernel<8, true>))
    SET_LDS((ffn_gemm_kernel8<2, true>))
    SET_LDS((ffn_gemm_kernel8<2, false>))
    SET_LDS((ffn_gemm_kernel8<4, true>))
    SET_LDS((ffn_gemm_kernel8<4, false>))
#undef SET_LDS
    return hipSuccess;
}

hipError_t launch_ffn_plan(const PlanArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(ffn_plan_kernel, dim3(PLAN_LISTS), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_down_combine(const moe_shape& s, const GemmArgs& args, const CombineArgs& c, bool out_fp32, hipStream_t st) {
    GemmArgs a = args;
    a.uniform_per = (s.T + 255) / 256;
    a.group_m = 8;
    a.shared_group = s.E;
    a.n_tiles = (s.H + 255) / 256;
    const dim3 grid((unsigned)(a.uniform_per * a.n_tiles));
    constexpr unsigned lds = COMBINE_LDS > NS * (256 + WROWS) * ROWB ? COMBINE_LDS : NS * (256 + WROWS) * ROWB;
#define DOWN_COMBINE(K_)                                                                                              \
    case K_:                                                                                                          \
        if (out_fp32) hipLaunchKernelGGL((ffn_down_combine_kernel<K_, true>), grid, dim3(256), lds, st, a, c);        \
        else hipLaunchKernelGGL((ffn_down_combine_kernel<K_, false>), grid, dim3(256), lds, st, a, c);                \
        break;
    switch (s.top_k) {
        DOWN_COMBINE(4)
        DOWN_COMBINE(5)
        DOWN_COMBINE(6)
        DOWN_COMBINE(7)
        DOWN_COMBINE(8)
        default: return hipErrorInvalidValue;
    }
#undef DOWN_COMBINE
    return hipGetLastError();
}

hipError_t launch_route_gemm(const GemmArgs& a, hipStream_t st) {
    const int cols = ((a.N + 63) / 64 + a.n_tiles - 1) / a.n_tiles;   // 64-expert blocks per tile (E <= 256)
    const dim3 grid((unsigned)(a.uniform_per * a.uniform_splits * a.n_tiles));
    const unsigned lds = NS * (a.uniform_tm + 64 * cols) * ROWB;
#define ROUTE(TI_, TJ_) hipLaunchKernelGGL((route_gemm_kernel<TI_, TJ_>), grid, dim3(256), lds, st, a)
#define ROUTE_COLS(TI_)                    \
    switch (cols) {                        \
        case 1: ROUTE(TI_, 1); break;      \
        case 2: ROUTE(TI_, 2); break;      \
        case 3: ROUTE(TI_, 3); break;      \
        case 4: ROUTE(TI_, 4); break;      \
        default: return hipErrorInvalidValue; \
    }
    if (a.uniform_tm == 128) ROUTE_COLS(2)
    else if (a.uniform_tm == 64) ROUTE_COLS(1)
    else return hipErrorInvalidValue;
#undef ROUTE_COLS
#undef ROUTE
    return hipGetLastError();
}

hipError_t launch_ffn_gemm(bool gated, const GemmArgs& a, const GemmConfig& cfg, hipStream_t st) {
    const dim3 grid((unsigned)(a.max_mtiles * a.n_tiles));
#define LAUNCH(KERNEL, THREADS) hipLaunchKernelGGL((KERNEL), grid, dim3(THREADS), MAX_LDS, st, a)
    if (cfg.waves == 8) {
        if (cfg.wave_rows == 4) {
            if (gated) LAUNCH((ffn_gemm_kernel8<4, true>), 512);
            else LAUNCH((ffn_gemm_kernel8<4, false>), 512);
        } else {
            if (gated) LAUNCH((ffn_gemm_kernel8<2, true>), 512);
            else LAUNCH((ffn_gemm_kernel8<2, false>), 512);
        }
    } else if (cfg.wave_rows == 2) {
        if (gated) LAUNCH((ffn_gemm_kernel<2, true>), 256);
        else LAUNCH((ffn_gemm_kernel<2, false>), 256);
    } else {
        if (gated) LAUNCH((ffn_gemm_kernel<1, true>), 256);
        else LAUNCH((ffn_gemm_kernel<1, false>), 256);
    }
#undef LAUNCH
    return hipGetLastError();
}

}  // namespace moe
