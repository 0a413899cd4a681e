// The m-tile lists of the two grouped GEMMs, built on the device from expert_offsets.
#pragma once
#include "common.h"

namespace moe {
namespace {

constexpr int PLAN_MAX_ROWS = 384;   // tallest m-tile
constexpr int PLAN_JOIN_ROWS = 64;   // a tail of up to that many rows joins its group's last full 256-row tile

// Exclusive prefix sums of three per-thread counters over the 256 threads of a workgroup, and
// their totals (every thread gets them): a wave-level scan, then the four wave sums through LDS.
__device__ __forceinline__ void block_scan3(int& a, int& b, int& c, int (&tot)[3], int (*wsum)[3], const int tid) {
    const int lane = tid & 63, w = tid >> 6;
    int ia = a, ib = b, ic = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int ta = __shfl_up(ia, d, 64), tb = __shfl_up(ib, d, 64), tc = __shfl_up(ic, d, 64);
        if (lane >= d) { ia += ta; ib += tb; ic += tc; }
    }
    if (lane == 63) { wsum[w][0] = ia; wsum[w][1] = ib; wsum[w][2] = ic; }
    __syncthreads();
    int oa = 0, ob = 0, oc = 0;
    tot[0] = tot[1] = tot[2] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < w) { oa += wsum[i][0]; ob += wsum[i][1]; oc += wsum[i][2]; }
        tot[0] += wsum[i][0]; tot[1] += wsum[i][1]; tot[2] += wsum[i][2];
    }
    __syncthreads();   // wsum may be written again
    a = oa + ia - a;
    b = ob + ib - b;
    c = oc + ic - c;
}

// How the rows of one group are cut into m-tiles for a tile height cap `tm`: tiles of `h` rows and a
// last one with the rest.  A group of two or three tiles is cut evenly, in steps of 32 rows: its
// tiles then run side by side, share the W panels they stream and finish together, where a short
// tail moved to the end of the list read them a second time (8x7B, 1511 tokens = 378 rows per
// expert: gate/up GEMM 740 -> 600 us, down 351 -> 300), and under a cap above 256 rows one of four (5003 tokens, 1250 rows =
// 4 x 320 instead of 3 x 352 and 194: down 940 -> 811).  A longer one is cut into full tiles and
// a tail.  A tail of at most 64 rows next to full 256-row tiles joins the last of them.
struct GroupCut {
    int cap, h, nfull, tail, joined;
    bool even;
};
__device__ __forceinline__ int div_small(const int a, const int b) {   // a / b for 0 <= a < 2^24, b >= 32: a short division
    int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
    if (q * b > a) --q;
    if ((q + 1) * b <= a) ++q;
    return q;
}
__device__ __forceinline__ GroupCut cut_group(const int rows, const int tm, const bool tall, const bool even) {
    GroupCut c;
    c.cap = c.h = tm;
    c.nfull = rows < (1 << 24) ? div_small(rows, tm) : rows / tm;
    c.tail = rows - c.nfull * tm;
    c.joined = tall && tm == 256 && c.nfull > 0 && c.tail <= PLAN_JOIN_ROWS ? c.tail : 0;
    c.tail -= c.joined;
    c.even = even && c.tail > 0 && c.nfull >= 1 && c.nfull <= (tm > 256 ? 3 : 2);
    if (c.even) {
        const int m = c.nfull + 1;
        c.h = ((m == 2 ? (rows + 1) >> 1 : m == 4 ? (rows + 3) >> 2 : (rows + 2) / 3) + 31) & ~31;
        c.nfull = m - (rows < m * c.h);   // (m - 1) * h < rows: rows > tm * (m - 1) >= 128 * (m - 1)
        c.tail = rows - c.nfull * c.h;
    }
    return c;
}

// The cut of one group for list `which` (0 gate/up, 1 down) with height cap tm; the cost of a list below and
// the list itself both use it.
// Shared experts next to short routed groups (up to about a thousand tokens): theirs are the longest
// tiles.  Down GEMM, where they walk all shared experts' K, and small gate/up launches: 128 rows at most unless
// the height is set by option (down GEMM, 64 experts + 2 shared, 300 tokens 96 -> 85 us, 500: 92 -> 90).  Gate/up:
// not cut evenly up to 512 tokens, so that the short rest goes last (500 tokens: 147 -> 143 us).
__device__ __forceinline__ GroupCut list_cut(const PlanArgs& p, const int which, const bool shared, const int rows, const int tm) {
    return cut_group(rows, shared && ((p.low_shared >> which) & 1) ? min(tm, 128) : tm, (which == 0 ? p.tall_up : p.tall_down) != 0,
                     !shared || which == 1 || p.T > 512);
}

// Height cap of a list's tiles, chosen from the call's real row counts.  What a tile costs per K
// sub-tile, in rows of matrix work (1.3 ns), is its height plus a constant for what it loads (a CU fills
// its LDS at about 44 GB/s): 290, and more where all CUs share the memory's bandwidth: 520 for a tile
// that streams its W panel alone, 340 next to another tile of its group.  (Uniform groups on the 8x7B layer: 0.72 us at
// 32 rows, 0.81 at 128, 1.01 at 256 with 1792 tiles; 0.42, 0.52 and 0.68 at 32, 128 and 256 rows
// with 128 tiles; 0.74 at 192 and 0.83 at 256 rows, two tiles to a panel.)  Above 256 rows the matrix cores take
// longer than the loads, 2.3 ns a row (8 experts, H = 6144, F = 16384, 16384 tokens, gate/up: 0.72 us at 256 rows, 0.88 at 320, 1.02
// at 384).  A launch costs its whole rounds of 256 tiles times the mean tile (of more than twelve the last one only half: by then the
// CUs are out of step), and no less than its longest tile.
//   short launches (up to two rounds of 256-row tiles, p.choose_* = 1): all eight caps.  With caps below 256 an expert of
//     250 rows is two tiles of 128: the down GEMM of eight such experts fills the chip with one round of 256 tiles instead
//     of half a round of 256-row ones (8x7B, 1000 tokens: 310 -> 268 us); with 352, one of 628 rows two tiles instead of three
//     (2500 tokens: one round instead of one and a half, 590 -> 424 us).
//   longer ones (2): 384, 352, 320 and 256 rows.  A taller tile moves fewer bytes from L2 to LDS per multiply-add, and its height
//     decides how the rounds come out: gate/up of 160 experts, 32768 tokens, 320 -> 384 rows 6230 -> 6110 us, down 256 -> 384
//     3450 -> 3260; 8 experts above 9190 -> 8910, 4860 -> 4740; 8x7B, 5003 tokens, down 256 -> 384 956 -> 825; 64 experts,
//     6000 tokens 491 -> 462, 282 -> 243.  Here a tile next to others of its group pays nothing extra for the panel (310 in all), a
//     lone one 500, and a tile of the shared experts' K-concatenated down GEMM counts as so many.  Groups just around a height
//     are what this has to get right (8x7B, gate/up, us): all of 350 to 380 rows, eight tiles of 384 rows per column 543 and
//     sixteen of 192 587; three of the eight above 384 rows, eleven tiles = 4.8 rounds 620 to 640 against 600 to 607, and the
//     even tiles stay.  (With half of the last round and 50 rows for the neighbour of a tile, the estimate took the
//     eleven, +7 %.)  Every height forced and timed, 633 launches of 280 to 32768 tokens, 2 to 160 experts: against the usual
//     height the chosen one takes 0.962 of the time (gate/up; the best of the four 0.954), 0.949 (down; 0.937), and no launch is
//     more than 3 % longer (one in 300 more than 1.5 %, which is what two timings of one launch differ by).  What another
//     height must gain by the estimate to be taken: 4 to 5 %, where 320 rows is the usual one (host, from 1200 rows per expert
//     on) 1.5 %.
constexpr int PLAN_CAPS = 8, PLAN_CAPS_LONG = 4;
__device__ constexpr int plan_cap(const int c) { return (c < 3 ? 384 : 352) - 32 * c; }   // 384, 352, 320, 256, 224, ... 128
// whether cap c is a candidate (3: as 1, for the wave grids that have no tiles above 256 rows)
__device__ constexpr bool plan_candidate(const int c, const int choose) { return choose == 1 || (choose == 2 ? c < PLAN_CAPS_LONG : choose == 3 && c >= 3); }

// What a list's tiles add up to under one cap.  n: tiles; alone: their group's only one; beside: next to others of
// their group (short launches); longest: highest tile.
struct ListSum {
    int n, alone, beside, longest;
    float sum;
};

// Groups first, first + step, ... of list `which`, cut with cap tm (shared experts of the down GEMM walk nseg0 segments).
__device__ __forceinline__ ListSum list_sum(const PlanArgs& p, const int which, const int* rows, const int ngroups, const int nseg0,
                                            const int tm, const int choose, const int first, const int step) {
    // cost of a tile of r rows, apart from what sharing the memory adds
    const int base = choose == 2 ? 310 : 290;
    auto tile = [=](const int r) { const int v = (r + 31) & ~31; return max(base + v, (v + 38) * 7 / 4); };
    ListSum s = {0, 0, 0, 0, 0.f};
    for (int g = first; g < ngroups; g += step) {
        const int r = rows[g];
        if (r == 0) continue;
        const GroupCut c = list_cut(p, which, p.Ns > 0 && (g == 0 || g > p.E), r, tm);
        const int m = c.nfull + (c.tail > 0);
        const int seg = g == 0 ? nseg0 : 1, weight = choose == 2 ? seg : 1;
        s.n += m * weight;
        if (m == 1) s.alone += weight;
        else if (choose != 2) s.beside += m;
        const int high = tile(m > 1 ? c.h : r);
        s.sum += (float)seg * (float)(c.nfull * high + (c.tail > 0 ? tile(c.tail) : 0) + (m > 1 ? c.joined : 0));
        s.longest = max(s.longest, high * seg);
    }
    return s;
}

__device__ __forceinline__ ListSum add_sums(const ListSum& a, const ListSum& b) {
    return {a.n + b.n, a.alone + b.alone, a.beside + b.beside, max(a.longest, b.longest), a.sum + b.sum};
}

__device__ __forceinline__ float list_cost(const ListSum& s, const int choose, const int n_tiles) {
    if (s.n == 0) return 0.f;
    const int tiles = s.n * n_tiles;
    const float busy = fminf(fmaxf((float)(tiles - 128) / 128.f, 0.f), 1.f);
    const float mean = (s.sum + busy * (50.f * s.beside + (choose == 2 ? 190.f : 230.f) * s.alone)) / (float)s.n;
    float rounds = (float)((tiles + 255) / 256);
    if (rounds > 12.f) rounds = 0.5f * (rounds + (float)tiles / 256.f + 0.5f);
    return fmaxf(rounds * mean, (float)s.longest);
}

// Builds an m-tile list (gate/up GEMM with tiles of up to tm_up rows, down GEMM with tm_down)
// from expert_offsets.  Group order: shared expert 0, routed experts, shared experts 1.. (the down
// GEMM takes the first two parts only: shared experts are concatenated along K there).
// cut_group says how a group's rows become tiles.  A tail higher than
// half a tile always stays with its group (on the variant that holds it, or the 256-row one after three
// full tiles and more: TILE_FULL).  tails_last = 0: the short tail, too, directly follows its group's tiles,
// which keeps the load-bound short tiles mixed with the compute-bound full ones (better when
// a launch has many rounds of tiles).  tails_last = 1: the short tails follow all other tiles,
// sorted by falling height, ties in group order, so a launch with few rounds ends on its
// smallest work items and its other tiles all take the same time (CUs that share operand
// panels in L2 stay in step).  n_run_* = number of entries listed in group order.
// One workgroup of 256 threads to a list (which: 0 gate/up, 1 down), side by side: the lists need nothing of each other, and
// both in one workgroup held up the launch around them.  `offsets`: E + 1 prefix sums in global memory or LDS.
constexpr int PLAN_LISTS = 2;
template <class Offsets>
__device__ __forceinline__ void plan_list(const PlanArgs& p, const int which, const Offsets offsets) {
    __shared__ int wsum[4][3];
    __shared__ int group_rows[256];
    __shared__ float cap_cost[PLAN_CAPS];
    const int tid = threadIdx.x;
    const int E = p.E, Ns = p.Ns;
    // group order: g = 0 -> shared 0 (if any), then routed 0..E-1, then shared 1..Ns-1
    const int ngroups = E + Ns;
    int row_begin = 0, rows = 0, group = 0, srow = -1;
    if (tid < ngroups) {
        int pos = tid;
        if (Ns > 0 && pos == 0) { group = E; rows = p.T; row_begin = 0; srow = 0; }
        else {
            if (Ns > 0) pos -= 1;
            if (pos < E) { group = pos; row_begin = offsets[pos]; rows = offsets[pos + 1] - row_begin; srow = -1; }
            else { const int s = pos - E + 1; group = E + s; rows = p.T; row_begin = 0; srow = s * p.t_pad; }
        }
        // a streamed pass covers routed experts [e_lo, e_hi) and, by shared_on, the shared experts
        if (group < E ? (group < p.e_lo || group >= p.e_hi) : !(p.shared_on >> which & (which == 0 ? 1 : 3))) rows = 0;
    }
    int tm = which == 0 ? p.tm_up : p.tm_down;
    const int choose = which == 0 ? p.choose_up : p.choose_down;
    // Routed groups that are one tile under every candidate cap leave nothing to choose, and the shared experts by themselves are
    // not worth the 3 us that it takes (small launches: p.low_shared; with one workgroup for both lists, 64 experts + 2 shared, 1500 tokens: the plan 12.8 us
    // with the choice and 9.1 without, the layer 350 and 347; 160 + 2, 3000 tokens: 15.6 and 9.4, 408 and 404).
    const int lowest = p.choose_up % 2 || p.choose_down % 2 ? 128 : 256;   // lowest cap: 2 has none below 256 rows
    if (choose && __syncthreads_or(group < E && rows > lowest)) {
        group_rows[tid] = rows;
        __syncthreads();
        const int c = tid >> 5;   // 32 lanes to a cap
        const int groups = which == 0 ? ngroups : (Ns > 0 ? E + 1 : E), nseg0 = which == 1 && Ns > 1 ? Ns : 1;
        ListSum sum = {0, 0, 0, 0, 0.f};
        if (plan_candidate(c, choose)) sum = list_sum(p, which, group_rows, groups, nseg0, plan_cap(c), choose, tid & 31, 32);
#pragma unroll
        for (int d = 1; d < 32; d <<= 1)
            sum = add_sums(sum, {__shfl_xor(sum.n, d, 64), __shfl_xor(sum.alone, d, 64), __shfl_xor(sum.beside, d, 64),
                                 __shfl_xor(sum.longest, d, 64), __shfl_xor(sum.sum, d, 64)});
        if ((tid & 31) == 0) cap_cost[c] = list_cost(sum, choose, which == 0 ? p.nt_up : p.nt_down);
        __syncthreads();
        // 256 rows, or 320 where the host says so, unless another height is clearly cheaper
        const int usual = choose == 2 && tm == 320 ? 2 : 3;
        float best = cap_cost[usual] * (usual == 2 ? 0.985f : (choose != 2 ? 0.97f : (which == 0 ? 0.96f : 0.95f)));
        tm = plan_cap(usual);
        for (int c = 0; c < PLAN_CAPS; ++c)
            if (plan_candidate(c, choose) && cap_cost[c] < best) { best = cap_cost[c]; tm = plan_cap(c); }
    }
    // Shared experts that only count: their tiles belong to another launch (launch_down_combine), and what is cut along K is decided as if they
    // were listed, so that the layer has the same bits either way.
    int apart = 0;
    if (which == 1 && (p.shared_on & 4)) {
        const GroupCut c = list_cut(p, 1, true, p.T, tm);
        apart = c.nfull + (c.tail > 0);
        if (group >= E) rows = 0;
    }
    TileDesc* descs = which == 0 ? p.descs_up : p.descs_down;
    const int tall = which == 0 ? p.tall_up : p.tall_down;
    const int last = which == 0 ? ngroups - 1 : (Ns > 0 ? E : E - 1);  // last group of this list
    const bool mine = tid <= last;
    const bool tails_last = (which == 0 ? p.tails_last_up : p.tails_last_down) != 0;
    const GroupCut cut = list_cut(p, which, group >= E, mine ? rows : 0, tm);
    const int nfull = cut.nfull, tail = cut.tail, joined = cut.joined, h = cut.h;
    const int blocks = (tail + 31) >> 5;   // 32-row blocks of the tail tile, 0 = none
    // A tail higher than half a tile takes nearly as long as a full tile, so it stays with its
    // group (keeps the group's W panels shared and the CUs in step); only a short tail is moved
    // to the end of the list.
    // (A shared expert's tail is not moved in a down list with K pieces: the pieces' partial
    // sums are reduced into y_perm, while shared rows belong to y_shared.)
    // (at most 128 rows: the K pieces' partial buffers hold SPLIT_TAIL_ROWS rows)
    const bool moved = tails_last && blocks > 0 && !cut.even && p.small_tiles && blocks * 64 <= min(cut.cap, 2 * SPLIT_TAIL_ROWS) &&
                       !(which == 1 && p.down_splits > 1 && group >= E);
    // tall_* = 2: the tall tile keeps its place in the group (it shares the W panels its
    // neighbours stream, which is the point when a group is only a few tiles).  tall_* = 1 and
    // tails_last: a tall tile takes longer than its neighbours and in a long launch puts the
    // CUs it runs on out of step for the rest of it, so it leaves the group order too: tall
    // tiles come first after the run region, one entry each, never cut along K.
    const bool tall_moved = tails_last && joined > 0 && tall == 1;
    const int nrun = nfull - (tall_moved ? 1 : 0) + (blocks > 0 && !moved);   // tiles listed in group order
    // Positions by prefix sums over the groups (at most 256, one per thread): tiles listed in
    // group order; tall tiles moved behind them; moved short tails, counted per height in
    // 32-row blocks (1..4), three 10-bit counters to a word.
    int base = nrun;
    int k2 = (tall_moved ? 1 : 0) | (moved && blocks == 1 ? 1 << 10 : 0) | (moved && blocks == 2 ? 1 << 20 : 0);
    int k3 = (moved && blocks == 3 ? 1 : 0) | (moved && blocks == 4 ? 1 << 10 : 0);
    int tot[3];
    block_scan3(base, k2, k3, tot, wsum, tid);
    const int n_run_s = tot[0], n_tall_s = tot[1] & 1023;
    const int cnt[5] = {0, (tot[1] >> 10) & 1023, (tot[1] >> 20) & 1023, tot[2] & 1023, (tot[2] >> 10) & 1023};
    const int pre[5] = {0, (k2 >> 10) & 1023, (k2 >> 20) & 1023, k3 & 1023, (k3 >> 10) & 1023};
    const int tails = cnt[1] + cnt[2] + cnt[3] + cnt[4];
    // Down list with K pieces: only the moved tails of at most p.split_max_blocks 32-row blocks are
    // cut (p.down_splits list entries each); the higher ones, which come first, stay whole.
    // Whether to cut at all is decided here, where the tile counts are known.  Pieces make a
    // launch faster in two cases only (measured on the Mixtral-shaped layer from 64 to 16384
    // tokens): when EVERY tile of the launch is a short tail (a few tokens per expert) and the
    // launch is bound by the walk along K, 0.42 us a sub-tile, and not by reading W at 5.8 TB/s and the 7 us of the
    // second launch: F / 32 * 0.42 > tiles * 512 F / 5.8e6 + 7, that is tiles <= 149 - 79000 / F =
    // p.split_room_tiles (whole -> cut, us: H = 2240, F = 7808, 63 tiles 97 -> 53; H = 4096, F = 14336, 128 tiles
    // 190 -> 162; H = 1216, F = 3072, 105 tiles 48 -> 42; but H = 2048, F = 2048, 128 tiles 30 -> 35; H = 6144,
    // F = 16384, 192 tiles 241 -> 279; H = 2560, F = 1664, 240 tiles 45 -> 72), and when the launch is
    // many rounds of tiles long (the tails at its end then finish sooner: -2 % on the
    // 16384-token, skewed workload).  In between, a launch of one to three rounds is as long
    // as its full tiles whatever happens to the tails, and pieces only add a round and
    // traffic (+6 ... +50 % measured).  p.split_rule_tiles: that many m-tiles or more count as
    // "many rounds"; 0: always cut.
    int n_whole = tails;
    bool cutting = which == 1 && p.down_splits > 1;
    if (cutting) {
        n_whole = 0;
        for (int b = p.split_max_blocks + 1; b <= 4; ++b) n_whole += cnt[b];
        const int others = n_run_s + n_tall_s + n_whole + apart;
        cutting = p.split_rule_tiles == 0 || (others == 0 && tails * p.nt_down <= p.split_room_tiles) || others + tails - n_whole >= p.split_rule_tiles;
        if (!cutting) n_whole = tails;
    }
    const int n_cut = tails - n_whole;
    if (tid == 0) {
        const int total = n_run_s + n_tall_s + n_whole + n_cut * (cutting ? p.down_splits : 1);
        // Tiles per XCD run (tile_order): 32, or 8 in a launch of a few rounds next to shared experts.
        // Theirs are the first and longest tiles of the list; in runs of 32 a few rounds of them
        // land on two or three XCDs, which then finish last (two shared experts next to 64 routed
        // ones, down GEMM: 1000 tokens 129 -> 95 us, 3001 tokens 174 -> 149 us).  Lists without them, of groups of streamed experts: 64 experts,
        // 1000 to 16384 tokens, and 160, 8000 and 32768, in groups of 8 to 32, layers in runs of 32 and of 8 within 0.2 % of each other.
        const int run = !p.xcd_remap ? 0 : (Ns > 0 && (p.shared_on >> which & 1) && total * (which == 0 ? p.nt_up : p.nt_down) <= 10 * 256 ? 8 : 32);
        if (which == 0) { p.plan->n_gate_up = total; p.plan->n_run_up = n_run_s; p.plan->xcd_run_up = run; }
        else { p.plan->n_down = total; p.plan->n_run_down = n_run_s; p.plan->n_split_tails = n_cut; p.plan->xcd_run_down = run; }
    }
    if (mine) {
        TileDesc d;
        d.group = group;
        d.srow = srow;
        const int once = p.mark_once && nfull + (blocks > 0) == 1 ? TILE_ONCE : 0;
        const int nlisted = nfull - (tall_moved ? 1 : 0);   // full tiles listed in group order
        // The rest of a group of four tiles and more keeps the full tiles' pace: a variant of 160 to 224 rows would put
        // its CUs out of step with those that share its panels (8x7B, 4782 tokens = 4.7 tiles per expert: +0.7 %).
        const int full = nfull >= 3 && blocks > 4 && blocks < 8 ? TILE_FULL : 0;
        for (int i = 0; i < nrun; ++i) {
            // entry nlisted (if any) is a tail that stays with its group; it starts after all full tiles
            const int at = i < nlisted ? i : nfull;
            d.row0 = row_begin + at * h;
            d.nrows = (min(h, rows - at * h) + ((at == nfull - 1 && !tall_moved) ? joined : 0)) | once | (at == nfull ? full : 0);
            descs[base + i] = d;
        }
        if (tall_moved) {
            const int before = k2 & 1023;   // tall tiles of the groups before this one
            d.row0 = row_begin + (nfull - 1) * h;
            d.nrows = (h + joined) | once;
            descs[n_run_s + before] = d;
        }
        if (moved) {
            // tails that come before this one: the higher ones, and those as high of earlier groups
            int rank = pre[blocks];
            for (int b = blocks + 1; b <= 4; ++b) rank += cnt[b];
            d.row0 = row_begin + nfull * h;
            // in more than one round it runs after the group's other tiles, if there are any; within one, next to them, and
            // the hint then costs as much as elsewhere (9 experts top-1 + 2 shared, H = 4544, F = 1920, 140 tokens:
            // gate/up 98 us with it, 73 without)
            const bool later = (n_run_s + n_tall_s) * (which == 0 ? p.nt_up : p.nt_down) > 256;
            d.nrows = tail | (p.mark_once && (nfull == 0 || later) ? TILE_ONCE : 0);
            const int tbase = n_run_s + n_tall_s;
            if (cutting && blocks <= p.split_max_blocks) {
                // one entry per K piece; the pieces' partial sums are added up after the launch
                const int q = rank - n_whole;   // falling height: the whole ones rank first
                for (int sp = 0; sp < p.down_splits; ++sp) {
                    d.srow = -2 - (q * p.down_splits + sp);
                    descs[tbase + n_whole + q * p.down_splits + sp] = d;
                }
                p.split_tails[q].row0 = d.row0;
                p.split_tails[q].nrows = tail;
            } else {
                descs[tbase + rank] = d;
            }
        }
    }
}

}  // namespace
}  // namespace moe
