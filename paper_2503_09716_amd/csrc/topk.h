// Softmax and top-k of a token whose logits sit in a row of 16 lanes.
#pragma once
#include "common.h"

namespace moe {
namespace {

// Butterfly step M of a wave-wide reduction: the value held by this lane's partner, the lane
// that differs from it in bit log2(M) and agrees in all higher bits.  Inside a row of 16 lanes
// the partner comes through the VALU's data-parallel-primitive path (quad permutes for M = 1, 2;
// half-row and row mirrors for M = 4, 8: lane i with 7-i, 15-i, which also flip the lower bits,
// and any partner with the same higher bits will do for a reduction); only M = 16, 32 go
// through the LDS crossbar, whose throughput per CU is what bounded the top-k kernels.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int M>
__device__ __forceinline__ int pair_i(int v) {
    if constexpr (M == 1) return dpp_move<0xB1>(v);        // quad_perm [1,0,3,2]
    else if constexpr (M == 2) return dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
    else if constexpr (M == 4) return dpp_move<0x141>(v);  // row_half_mirror
    else if constexpr (M == 8) return dpp_move<0x140>(v);  // row_mirror
    else return __shfl_xor(v, M, 64);
}
template <int M>
__device__ __forceinline__ float pair_f(float v) {
    return __int_as_float(pair_i<M>(__float_as_int(v)));
}

__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, pair_f<1>(v));
    v = fmaxf(v, pair_f<2>(v));
    v = fmaxf(v, pair_f<4>(v));
    v = fmaxf(v, pair_f<8>(v));
    return v;
}
__device__ __forceinline__ float row16_sum(float v) {
    v += pair_f<1>(v);
    v += pair_f<2>(v);
    v += pair_f<4>(v);
    v += pair_f<8>(v);
    return v;
}
__device__ __forceinline__ uint32_t row16_max(uint32_t v) {
    v = max(v, (uint32_t)pair_i<1>((int)v));
    v = max(v, (uint32_t)pair_i<2>((int)v));
    v = max(v, (uint32_t)pair_i<4>((int)v));
    v = max(v, (uint32_t)pair_i<8>((int)v));
    return v;
}
__device__ __forceinline__ int row16_min(int v) {
    v = min(v, pair_i<1>(v));
    v = min(v, pair_i<2>(v));
    v = min(v, pair_i<4>(v));
    v = min(v, pair_i<8>(v));
    return v;
}

// A logit as an unsigned integer of the same order (-0 as +0).  NaN comes below everything else (1); 0 is left for "not a candidate".
constexpr uint32_t KEY_OF_NAN = 1u, KEY_OF_ZERO = 0x80000000u;
__device__ __forceinline__ uint32_t logit_key(const float v) {
    const uint32_t u = __float_as_uint(v + 0.f);
    return v == v ? ((int32_t)u < 0 ? ~u : u | 0x80000000u) : KEY_OF_NAN;
}
__device__ __forceinline__ float key_logit(const uint32_t k) {
    return __uint_as_float(k == KEY_OF_NAN ? 0x7fc00000u : (k & 0x80000000u ? k & 0x7fffffffu : ~k));
}

// Softmax over all experts + top-k (k <= 16) for the token held by one ROW of 16 lanes: the lane
// with row index c holds the logits of experts c, c+16, ... in v[] (-inf past E); a wavefront
// finishes four tokens at once.  Selection is on the logits (ties -> lower expert id), so rounding
// in exp / division can never change it: per pick the largest key of the row, then the lowest
// expert that holds it, four butterfly steps each on the VALU's DPP path; the pick's weight is computed from
// its logit once all are known.  (Against butterflies that carried
// (logit, expert, exp) and compared pairs, and partial logits added one load at a time, the route stage: 64 experts top-6, 1 token
// 11.9 -> 9.2 us, 3001: 20.8 -> 18.3; 160 experts, 1 token 17.0 -> 11.3, 2000: 35.7 -> 30.4.)
// Lane j of the row ends up with the j-th pick: my_e, my_w (meaningful for row < k).
// WIDE: the lane holds experts 4c..4c+3, 64+4c..64+4c+3, ... instead (what 16-byte loads of a
// row of logits deliver); either way its experts ascend with i.
template <bool WIDE>
__device__ __forceinline__ int row16_expert(const int row, const int i) {
    return WIDE ? row * 4 + (i & 3) + 64 * (i >> 2) : row + 16 * i;
}
template <int NV, bool WIDE = false>
__device__ __forceinline__ void route_select_row16(const float (&v)[NV], const int row, const int E, const int k, const int renorm,
                                                   const float scale, int& my_e, float& my_w) {
    float m = -INFINITY;
    uint32_t key[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        m = fmaxf(m, v[i]);
        key[i] = row16_expert<WIDE>(row, i) < E ? logit_key(v[i]) : 0u;
    }
    m = row16_max(m);
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) z += expf(v[i] - m);   // exp(-inf) = 0 for padded experts
    const float rz = 1.0f / row16_sum(z);
    uint32_t my_key = KEY_OF_ZERO;
    my_e = 0;
    for (int j = 0; j < k; ++j) {
        uint32_t best = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) best = max(best, key[i]);
        best = row16_max(best);
        int e = 0x7fffffff;
#pragma unroll
        for (int i = NV - 1; i >= 0; --i) e = key[i] == best ? row16_expert<WIDE>(row, i) : e;
        e = row16_min(e);
#pragma unroll
        for (int i = 0; i < NV; ++i) key[i] = row16_expert<WIDE>(row, i) == e ? 0u : key[i];
        if (row == j) { my_e = e; my_key = best; }
    }
    my_w = expf(key_logit(my_key) - m) * rz;
    const float wsum = row16_sum(row < k ? my_w : 0.f);
    if (renorm) my_w = my_w / wsum;
    my_w *= scale;
}

template <int NV, bool WIDE = false>
__device__ __forceinline__ void route_finish_row16(const float (&v)[NV], const int row, const int tok, const bool valid,
                                                   const int E, const int k, const int renorm, const float scale,
                                                   int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                                   float* __restrict__ logits_out) {
    if (logits_out && valid) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int e = row16_expert<WIDE>(row, i);
            if (e < E) logits_out[(size_t)tok * E + e] = v[i];
        }
    }
    int e;
    float w;
    route_select_row16<NV, WIDE>(v, row, E, k, renorm, scale, e, w);
    if (valid && row < k) {
        idx_out[(size_t)tok * k + row] = e;
        w_out[(size_t)tok * k + row] = w;
    }
}

// The logits of token t from `splits` partial matrices [splits][T][EP], added in order, plus the bias.  Lane c of a
// row of 16 takes experts 4c..4c+3 of every 64 as one 16-byte load per matrix (NB = blocks of 64 experts).
template <int NB>
__device__ __forceinline__ void sum_logits_row16(float (&v)[4 * NB], const float* __restrict__ partial, const int splits, const int T, const int EP,
                                                 const int E, const float* __restrict__ bias, const int t, const int row) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int e0 = row * 4 + 64 * b;
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
        if (e0 < EP)   // EP is a multiple of 32: the four values are all inside the row or all outside
#pragma unroll 4
            for (int s = 0; s < splits; ++s) a += *reinterpret_cast<const f32x4*>(partial + ((size_t)s * T + t) * EP + e0);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[4 * b + q] = e0 + q < E ? a[q] + (bias ? bias[e0 + q] : 0.f) : -INFINITY;
    }
}

// One wavefront: tokens 4 * quad .. 4 * quad + 3.
template <int NB>
__device__ __forceinline__ void topk_row16(const float* __restrict__ partial, const int splits, const int T, const int EP, const int E, const int k,
                                           const float* __restrict__ bias, const int renorm, const float scale, const int quad, const int lane,
                                           int32_t* __restrict__ idx_out, float* __restrict__ w_out, float* __restrict__ logits_out) {
    const int row = lane & 15, tok = quad * 4 + (lane >> 4);
    float v[4 * NB];
    sum_logits_row16<NB>(v, partial, splits, T, EP, E, bias, min(tok, T - 1), row);   // rows past the end redo the last token and write nothing
    route_finish_row16<4 * NB, true>(v, row, tok, tok < T, E, k, renorm, scale, idx_out, w_out, logits_out);
}

}  // namespace
}  // namespace moe
