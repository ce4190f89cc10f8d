// Selection of the k largest scores of a row held in registers: the device half shared by the
// top-k kernel and by the gather of a small retrieval.
#pragma once

#include "oqm_device.h"

namespace oqm {

// Larger float <=> larger unsigned key, never 0 (the key of an absent entry); -0 and +0 map to
// the same key.
__device__ __forceinline__ uint32_t orderable(float s) {
    const uint32_t u = __float_as_uint(s + 0.0f);
    return max(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u), 1u);
}

// Number of lanes below this one in the ballot `b`.
__device__ __forceinline__ uint32_t rank_in(uint64_t b) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

// WAVES waves hold the keys of one row, KEYS per lane: wave w, register c, lane l is entry
// (w * KEYS + c) * 64 + l of the row (absent ones hold key 0; at least k_eff are present).  Calls emit(rank, entry)
// in the lane of each of the k_eff largest keys, ranks 0 .. k_eff - 1 in ascending entry order; of equal keys the
// lowest entries are taken.  The k-th largest key is built bit by bit from the top: a bit stays set if at
// least k keys reach the candidate, and the search ends early when exactly k do.  A count is
// KEYS ballots and scalar population counts; with one wave there is no barrier and no LDS at all,
// with several each count is one exchange through `slots` (two alternating sets of WAVES words).
template <int WAVES, int KEYS, typename EMIT>
__device__ __forceinline__ void select_largest(const uint32_t (&key)[KEYS], int k_eff, int wave, int lane,
                                               uint32_t (*slots)[WAVES], EMIT emit) {
    int phase = 0;
    // sum over aligned sets of WAVES lanes (DPP), as a scalar
    auto lanes_sum = [](uint32_t v) -> uint32_t {
        if constexpr (WAVES >= 2) v += dpp_u32<0xB1>(v);
        if constexpr (WAVES >= 4) v += dpp_u32<0x4E>(v);
        if constexpr (WAVES >= 8) v += dpp_u32<0x141>(v);
        if constexpr (WAVES >= 16) v += dpp_u32<0x140>(v);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };
    // every wave's count, in lane w of each aligned set of WAVES lanes
    auto exchange = [&](uint32_t mine) -> uint32_t {
        if (lane == 0) slots[phase][wave] = mine;
        __syncthreads();
        const uint32_t v = slots[phase][lane & (WAVES - 1)];
        phase ^= 1;
        return v;
    };
    auto across = [&](uint32_t mine) -> uint32_t {
        if constexpr (WAVES == 1) return mine;
        else return lanes_sum(exchange(mine));
    };
    uint32_t thr = 0;   // the k-th largest key; only keys above it once `exact`
    bool exact = false;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)(thr | (1u << bit)));
        uint32_t mine = 0;
#pragma unroll
        for (int c = 0; c < KEYS; ++c) mine += (uint32_t)__popcll(__ballot(key[c] >= cand));
        const uint32_t cnt = across(mine);
        if (cnt >= (uint32_t)k_eff) thr = cand;
        if (cnt == (uint32_t)k_eff) {
            exact = true;
            break;
        }
    }
    if (exact) thr -= 1u;   // "above thr" is now exactly the chosen set (cand >= 1)

    uint32_t gt_mine = 0, eq_mine = 0;
#pragma unroll
    for (int c = 0; c < KEYS; ++c) {
        gt_mine += (uint32_t)__popcll(__ballot(key[c] > thr));
        eq_mine += (uint32_t)__popcll(__ballot(key[c] == thr));
    }
    uint32_t gt_all = gt_mine, base_g = 0, base_e = 0;   // in all waves; in the waves before this one
    if constexpr (WAVES > 1) {
        const uint32_t g = exchange(gt_mine), e = exchange(eq_mine);
        const bool earlier = (lane & (WAVES - 1)) < wave;
        gt_all = lanes_sum(g);
        base_g = lanes_sum(earlier ? g : 0u);
        base_e = lanes_sum(earlier ? e : 0u);
    }
    const uint32_t need = (uint32_t)k_eff - gt_all;   // entries equal to thr to take, lowest first
#pragma unroll
    for (int c = 0; c < KEYS; ++c) {
        const int i = (wave * KEYS + c) * 64 + lane;
        const bool gt = key[c] > thr;
        const bool eq = key[c] == thr;
        const uint64_t bg = __ballot(gt), be = __ballot(eq);
        const uint32_t og = base_g + rank_in(bg), oe = base_e + rank_in(be);
        if (gt) emit(og + min(oe, need), i);
        else if (eq && oe < need) emit(og + oe, i);
        base_g += (uint32_t)__popcll(bg);
        base_e += (uint32_t)__popcll(be);
    }
}

// The keys of a row of n scores for select_largest.
template <int KEYS>
__device__ __forceinline__ void load_keys_of_row(const float* __restrict__ s, int n, int wave, int lane,
                                                 uint32_t (&key)[KEYS]) {
    float x[KEYS];
#pragma unroll
    for (int c = 0; c < KEYS; ++c) x[c] = s[(uint32_t)min((wave * KEYS + c) * 64 + lane, n - 1)];
#pragma unroll
    for (int c = 0; c < KEYS; ++c) {
        asm volatile("" : "+v"(x[c]));  // all loads in flight before the first is used (the compiler would branch around each)
        key[c] = (wave * KEYS + c) * 64 + lane < n ? orderable(x[c]) : 0u;
    }
}

}  // namespace oqm
