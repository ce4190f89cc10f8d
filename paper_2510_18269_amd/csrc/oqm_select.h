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
// lowest entries are taken.  The k-th largest key is built from the top: the largest extension of it that at
// least k keys reach is taken, and the search ends early when exactly k do.  A count is
// KEYS ballots and scalar population counts.  One wave settles a bit at a time, with no barrier and no
// LDS at all; several exchange their counts through `slots` (two alternating sets of two words a wave), which
// is most of a step, so a step of theirs settles two bits with three counts.  Equal scores at the
// threshold take all steps: 28 rows of 1024 scores with each score five times over 6.9 us, 7.8 with steps of one bit.
template <int WAVES, int KEYS, typename EMIT>
__device__ __forceinline__ void select_largest(const uint32_t (&key)[KEYS], int k_eff, int wave, int lane,
                                               uint32_t (*slots)[2 * WAVES], EMIT emit) {
    int phase = 0;
    // sum over aligned sets of WAVES lanes (DPP), as a scalar
    auto lanes_sum = [](uint32_t v) -> uint32_t {
        if constexpr (WAVES >= 2) v += dpp_u32<0xB1>(v);
        if constexpr (WAVES >= 4) v += dpp_u32<0x4E>(v);
        if constexpr (WAVES >= 8) v += dpp_u32<0x141>(v);
        if constexpr (WAVES >= 16) v += dpp_u32<0x140>(v);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };
    // two words of every wave, in lane w of each aligned set of WAVES lanes
    auto exchange = [&](uint32_t& x, uint32_t& y) {
        if (lane == 0) {
            slots[phase][2 * wave] = x;
            slots[phase][2 * wave + 1] = y;
        }
        __syncthreads();
        x = slots[phase][2 * (lane & (WAVES - 1))];
        y = slots[phase][2 * (lane & (WAVES - 1)) + 1];
        phase ^= 1;
    };
    // keys of this wave that reach `cand`
    auto reach = [&](uint32_t cand) -> uint32_t {
        uint32_t mine = 0;
#pragma unroll
        for (int c = 0; c < KEYS; ++c) mine += (uint32_t)__popcll(__ballot(key[c] >= cand));
        return mine;
    };
    uint32_t thr = 0;   // the k-th largest key; only keys above it once `exact`
    bool exact = false;
    constexpr int STEP = WAVES == 1 ? 1 : 2;   // bits settled per count
    for (int bit = 32 - STEP; bit >= 0; bit -= STEP) {
        const uint32_t one = 1u << bit;
        const uint32_t c1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(thr | one));
        uint32_t cand = c1, cnt;
        if constexpr (STEP == 1) {
            cnt = reach(c1);
        } else {
            const uint32_t c2 = c1 + one, c3 = c2 + one;
            uint32_t n12 = reach(c1) | reach(c2) << 16, n3 = reach(c3);   // at most 4096 each
            exchange(n12, n3);
            n12 = lanes_sum(n12);
            cnt = n12 & 0xffffu;
            n3 = lanes_sum(n3);
            if ((n12 >> 16) >= (uint32_t)k_eff) {
                cand = c2;
                cnt = n12 >> 16;
            }
            if (n3 >= (uint32_t)k_eff) {
                cand = c3;
                cnt = n3;
            }
        }
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
        uint32_t g = gt_mine, e = eq_mine;
        exchange(g, e);
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
