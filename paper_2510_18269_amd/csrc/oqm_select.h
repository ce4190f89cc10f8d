// Selection of the k largest scores of a row held in registers: the device half shared by the
// top-k kernel and by the gather of a small retrieval.
#pragma once

#include <type_traits>

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

// Inclusive sum over the lanes of a wave up to this one.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    auto step = [&](auto ctrl, auto rows) {
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});  // row_shr:1, 2, 4, 8
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});  // row_bcast:15 into rows 1 and 3
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});  // row_bcast:31 into rows 2 and 3
    return v;
}

constexpr int kHistCopies = 4;        // words per bin: lanes that add to one bin take turns
constexpr uint32_t kSelectList = 16;  // keys that are ranked in less time than another digit takes

// Memory that the waves of select_largest share.
template <int WAVES>
struct alignas(16) SelectScratch {
    uint32_t hist[2][256 * kHistCopies];
    uint32_t list[kSelectList];
    uint32_t slots[2][2 * WAVES];
    uint32_t listed;
};

// WAVES waves hold the keys of one row, KEYS per lane: wave w, register c, lane l is entry
// (w * KEYS + c) * 64 + l of the row (absent ones hold key 0; more than k_eff are present).  Calls emit(rank, entry)
// in the lane of each of the k_eff largest keys, ranks 0 .. k_eff - 1 in ascending entry order; of equal keys the
// lowest entries are taken.
// The k-th largest key is found from the top, eight bits at a time: the keys that share its upper digits are counted by their next one
// in LDS, and every wave scans the 256 counts by itself, so a digit costs a barrier or none.  The search ends early when a range
// is chosen whole, when it is down to 16 keys (these are listed, and every wave ranks the list by itself), or when a digit has not divided it and all
// its keys are equal (a camera that does not move).  Bound by the latency of its serial steps: two digits and the list at random scores.  Lanes that
// add to one word take their turns, hence four words a bin.  28 rows in a graph, this / two bits a barrier by ballots: 200
// scores 2.9 / 3.0 us, 1024 3.7 / 5.0, 2000 3.9 / 6.1, 3600 5.6 / 7.4; 1024 equal ones 3.6 / 4.7, 4096 6.2 / 7.0 (one word a bin 10.8), each of 1024 five
// times 3.8 / 5.3, 777 with 60 of each 4.1 / 5.5.  One word a bin and a test of each register for lanes that all share a bin: 3.9 at 1024, 6.4 at 3600.
// Ballots end sooner where a few high scores stand apart, and start without clearing counts: one row, the first 1 to 4 of 300 to 777 scores 3.0 to 3.6 / 2.7 to
// 3.1, of up to 256 2.5 to 3.0 / 2.2 to 3.0; the first 16 or 64 of 300 to 777 3.4 / 4.4 to 5.0.
template <int WAVES, int KEYS, typename EMIT>
__device__ __forceinline__ void select_largest(const uint32_t (&key)[KEYS], int k_eff, int wave, int lane,
                                               SelectScratch<WAVES>* shared, EMIT emit) {
    // what the waves have written is read by all; one wave's LDS operations are in order anyway
    auto sync = [] {
        if constexpr (WAVES > 1) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    };
    // sum over aligned sets of WAVES lanes (DPP), as a scalar
    auto lanes_sum = [](uint32_t v) -> uint32_t {
        if constexpr (WAVES >= 2) v += dpp_u32<0xB1>(v);
        if constexpr (WAVES >= 4) v += dpp_u32<0x4E>(v);
        if constexpr (WAVES >= 8) v += dpp_u32<0x141>(v);
        if constexpr (WAVES >= 16) v += dpp_u32<0x140>(v);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };
    int phase = 0;
    // two words of every wave, in lane w of each aligned set of WAVES lanes
    auto exchange = [&](uint32_t& x, uint32_t& y) {
        if constexpr (WAVES > 1) {
            if (lane == 0) {
                shared->slots[phase][2 * wave] = x;
                shared->slots[phase][2 * wave + 1] = y;
            }
            __syncthreads();
            x = shared->slots[phase][2 * (lane & (WAVES - 1))];
            y = shared->slots[phase][2 * (lane & (WAVES - 1)) + 1];
            phase ^= 1;
        }
    };
    auto clear = [&](int digit, int n) {
        u32x4* const h = reinterpret_cast<u32x4*>(shared->hist[digit & 1]);
        for (int i = wave * 64 + lane; i < n * 64 * kHistCopies; i += 64 * WAVES) h[i] = u32x4{0u, 0u, 0u, 0u};
    };
    clear(0, 2);
    if (wave == 0 && lane == 0) shared->listed = 0u;
    sync();

    uint32_t thr = 0;   // the k-th largest key; only keys above it once `exact`
    uint32_t hi = 0;    // keys above the range that is looked at
    uint32_t before = 64 * KEYS * WAVES, unequal = 0;  // keys in it; the last size that did not hold one value only
    bool exact = false;
    for (int digit = 0; digit < 4; ++digit) {
        const int shift = 24 - 8 * digit;
        uint32_t* const hist = shared->hist[digit & 1];
        if (digit >= 2) {  // rarely
            clear(digit, 1);
            sync();
        }
#pragma unroll
        for (int c = 0; c < KEYS; ++c)
            if (digit == 0 || (key[c] ^ thr) >> (shift + 8) == 0)
                atomicAdd(&hist[((key[c] >> shift) & 255u) * kHistCopies + (lane & (kHistCopies - 1))], 1u);
        sync();
        // lane l owns the bins 252 - 4 l .. 255 - 4 l, so that the scan runs from the largest digit down
        uint32_t n[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const u32x4 w = reinterpret_cast<const u32x4*>(hist)[252 - 4 * lane + b];
            n[b] = w[0] + w[1] + w[2] + w[3];
        }
        const uint32_t want = (uint32_t)k_eff - hi;
        const uint32_t incl = wave_scan(n[0] + n[1] + n[2] + n[3]);
        const uint32_t c3 = incl - n[0] - n[1] - n[2], c2 = c3 + n[2], c1 = c2 + n[1];  // keys down to bin 3, 2, 1 of the four
        const uint32_t excl = c3 - n[3];
        uint32_t bin = 255u - 4u * (uint32_t)lane, above = excl, range = n[3];
        if (want > c3) bin -= 1u, above = c3, range = n[2];
        if (want > c2) bin -= 1u, above = c2, range = n[1];
        if (want > c1) bin -= 1u, above = c1, range = n[0];
        const int at = __builtin_ctzll(__ballot(excl < want && want <= incl));  // exactly one lane
        thr |= (uint32_t)__builtin_amdgcn_readlane((int)bin, at) << shift;
        hi += (uint32_t)__builtin_amdgcn_readlane((int)above, at);
        range = (uint32_t)__builtin_amdgcn_readlane((int)range, at);
        if (hi + range == (uint32_t)k_eff) {
            exact = true;
            break;
        }
        if (shift == 0) break;
        if (range <= kSelectList) {
#pragma unroll
            for (int c = 0; c < KEYS; ++c)
                if ((key[c] ^ thr) >> shift == 0) shared->list[atomicAdd(&shared->listed, 1u)] = key[c];
            sync();
            const uint32_t left = (uint32_t)k_eff - hi;
            const uint32_t x = shared->list[min((uint32_t)lane, range - 1u)];
            uint32_t greater = 0, reach = 0;  // listed keys above this lane's, and at least it
            for (uint32_t j = 0; j < range; ++j) {
                const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)j);
                greater += y > x;
                reach += y >= x;
            }
            thr = (uint32_t)__builtin_amdgcn_readlane((int)x, __builtin_ctzll(__ballot(greater < left && reach >= left)));
            break;
        }
        if (digit > 0 && range == before && range != unequal) {  // uniform, like the counts
            uint32_t first = 0, same = 1;  // a key of this wave in the range (0: none), and whether all are it
#pragma unroll
            for (int c = 0; c < KEYS; ++c) {
                const uint64_t in = __ballot((key[c] ^ thr) >> shift == 0);
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
        before = range;
    }
    if (exact) thr -= 1u;   // "above thr" is now exactly the chosen set (thr >= 1: a present key reaches it)

    uint32_t gt_all = 0, base_g = 0, base_e = 0;  // keys above thr: in all waves, in the waves before this one; keys equal to it there
    {
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
