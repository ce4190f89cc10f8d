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

constexpr uint32_t kSelectList = 16;  // keys that are ranked in less time than two more steps take

// Memory that the waves of select_largest share (one wave uses none).
template <int WAVES>
struct SelectScratch {
    uint32_t slots[2][2 * WAVES];
    uint32_t list[kSelectList];
};

// WAVES waves hold the keys of one row, KEYS per lane: wave w, register c, lane l is entry
// (w * KEYS + c) * 64 + l of the row (absent ones hold key 0; more than k_eff are present).  Calls emit(rank, entry)
// in the lane of each of the k_eff largest keys, ranks 0 .. k_eff - 1 in ascending entry order; of equal keys the
// lowest entries are taken.  The k-th largest key is built from the top: the largest extension of it that at
// least k keys reach is taken, and the search ends early when exactly k do.  A count is
// KEYS ballots and scalar population counts.  One wave settles a bit at a time, with no barrier and no
// LDS at all.  Several exchange their counts through `slots` (two alternating sets of two words a wave), which
// is most of a step (0.28 us), so a step of theirs settles two bits with three counts; once the range that holds
// the k-th key is down to 16 keys these are listed and every wave ranks the list by itself.  Scores that occur
// several times (a camera that does not move) never let the search end with exactly k, and 16 steps are slower
// than the radix select of oqm_topk.hip: they end on the list, or, if more than 16 are equal, by the comparison of a
// range that a step inside the mantissa has not divided with one of its keys.  28 rows of 1024 scores, this / without
// list and comparison / radix select: all different 5.3 / 5.2 / 5.9 us, each five times over 5.6 / 6.7 / 5.9, all
// equal 4.8 / 6.5 / 8.6.  Listing at 64 keys: 5.5 / 5.6 / 4.9, and 7.2 instead of 6.2 us at 777 scores with 60 of each.
template <int WAVES, int KEYS, typename EMIT>
__device__ __forceinline__ void select_largest(const uint32_t (&key)[KEYS], int k_eff, int wave, int lane,
                                               SelectScratch<WAVES>* shared, EMIT emit) {
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
            shared->slots[phase][2 * wave] = x;
            shared->slots[phase][2 * wave + 1] = y;
        }
        __syncthreads();
        x = shared->slots[phase][2 * (lane & (WAVES - 1))];
        y = shared->slots[phase][2 * (lane & (WAVES - 1)) + 1];
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
    bool exact = false, counted = false;
    uint32_t gt_all = 0, base_g = 0, base_e = 0;   // keys above thr: in all waves; in the waves before this one, and keys equal to it there
    if constexpr (WAVES == 1) {
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)(thr | 1u << bit));
            const uint32_t cnt = reach(cand);
            if (cnt >= (uint32_t)k_eff) thr = cand;
            if (cnt == (uint32_t)k_eff) {
                exact = true;
                break;
            }
        }
    } else {
        const bool earlier = (lane & (WAVES - 1)) < wave;
        uint32_t lo = 64 * KEYS * WAVES, hi = 0;  // keys from thr on; keys above the range [thr, thr + 2^bit)
        uint32_t lo_w = 64 * KEYS, hi_w = 0;      // lane w: of these those of wave w
        uint32_t unequal = 0;                     // size of the last range that did not hold one value only
        for (int bit = 30; bit >= 0; bit -= 2) {
            const uint32_t one = 1u << bit, before = lo - hi;
            const uint32_t c1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(thr | one)), c2 = c1 + one, c3 = c2 + one;
            uint32_t w12 = reach(c1) | reach(c2) << 16, w3 = reach(c3);  // at most 4096 each
            exchange(w12, w3);
            const uint32_t n12 = lanes_sum(w12), n1 = n12 & 0xffffu, n2 = n12 >> 16, n3 = lanes_sum(w3);
            const uint32_t w1 = w12 & 0xffffu, w2 = w12 >> 16;
            if (n3 >= (uint32_t)k_eff) {
                thr = c3, lo = n3, lo_w = w3;
            } else if (n2 >= (uint32_t)k_eff) {
                thr = c2, lo = n2, lo_w = w2, hi = n3, hi_w = w3;
            } else if (n1 >= (uint32_t)k_eff) {
                thr = c1, lo = n1, lo_w = w1, hi = n2, hi_w = w2;
            } else {
                hi = n1, hi_w = w1;
            }
            if (lo == (uint32_t)k_eff) {
                exact = true;
                break;
            }
            const uint32_t range = lo - hi;
            if (bit > 0 && range <= kSelectList) {  // uniform, like all that follows from the exchanged counts
                const uint32_t first = lanes_sum(earlier ? lo_w - hi_w : 0u);  // this wave's place in the list
                uint32_t at = first;
#pragma unroll
                for (int c = 0; c < KEYS; ++c) {
                    const bool in = key[c] - thr < one;
                    const uint64_t b = __ballot(in);
                    if (in) shared->list[at + rank_in(b)] = key[c];
                    at += (uint32_t)__popcll(b);
                }
                __syncthreads();
                const uint32_t x = (uint32_t)lane < range ? shared->list[lane] : 0u;
                uint32_t above = 0;  // listed keys above this lane's
                for (uint32_t j = 0; j < range; j += 8) {  // padded with zeros, which are above none
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) above += (uint32_t)__builtin_amdgcn_readlane((int)x, (int)(j + u)) > x;
                }
                const uint32_t want = (uint32_t)k_eff - hi;
                // The k-th key: of all with fewer than `want` above them the one with the most, want - 1 unless it occurs
                // again.  Lanes past the list have at least `want` keys above them.
                uint64_t eq = __ballot(above == want - 1);
                if (!eq) {
                    uint32_t most = 0;
                    for (uint64_t rest = __ballot(above < want); rest; rest = __ballot(above > most && above < want))
                        most = (uint32_t)__builtin_amdgcn_readlane((int)above, __builtin_ctzll(rest));
                    eq = __ballot(above == most);
                }
                thr = (uint32_t)__builtin_amdgcn_readlane((int)x, __builtin_ctzll(eq));
                const uint64_t gt = __ballot(x > thr), front = (1ull << first) - 1;
                gt_all = hi + (uint32_t)__popcll(gt);
                base_g = lanes_sum(earlier ? hi_w : 0u) + (uint32_t)__popcll(gt & front);
                base_e = (uint32_t)__popcll(eq & front);
                counted = true;
                break;
            }
            if (bit > 0 && bit < 22 && range == before && range != unequal) {  // uniform, like the counts
                uint32_t first = 0, same = 1;  // a key of this wave in the range (0: none), and whether all are it
#pragma unroll
                for (int c = 0; c < KEYS; ++c) {
                    const uint64_t in = __ballot(key[c] - thr < one);
                    if (in && !first) first = (uint32_t)__builtin_amdgcn_readlane((int)key[c], __builtin_ctzll(in));
                    if (__ballot(key[c] == first) & in ^ in) same = 0;
                }
                exchange(first, same);
                const uint64_t some = __ballot(first != 0);  // the range holds a present key: some wave has one
                const uint32_t value = (uint32_t)__builtin_amdgcn_readlane((int)first, __builtin_ctzll(some));
                if (!__ballot(same == 0 || (first != 0 && first != value))) {
                    thr = value;
                    break;
                }
                unequal = range;
            }
        }
    }
    if (exact) thr -= 1u;   // "above thr" is now exactly the chosen set (cand >= 1)

    if (!counted) {
        uint32_t g = 0, e = 0;
#pragma unroll
        for (int c = 0; c < KEYS; ++c) {
            g += (uint32_t)__popcll(__ballot(key[c] > thr));
            e += (uint32_t)__popcll(__ballot(key[c] == thr));
        }
        gt_all = g;
        if constexpr (WAVES > 1) {
            exchange(g, e);
            const bool earlier = (lane & (WAVES - 1)) < wave;
            gt_all = lanes_sum(g);
            base_g = lanes_sum(earlier ? g : 0u);
            base_e = lanes_sum(earlier ? e : 0u);
        }
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
