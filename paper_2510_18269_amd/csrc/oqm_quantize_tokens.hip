// Store step with the quantization axis of the paper's Eq. 9: one (scale, zero) pair per
// head and channel, taken over the G tokens of the frame-group (Sec. 3.4, Eq. 8 and Eq. 9),
// plus nibble packing and the summary key, for one head tile per workgroup.
//
// Both forms: a 1-D grid, first the K tiles, then the V tiles, in the order of a contiguous input, so that one dense stream of
// addresses is read at a time and the workgroups that also sum start first.  Keys averaged over another tensor
// have workgroups of their own in front of those (one pass over that tensor, as many rows in flight as the
// tiles' own), instead of a second pass by the workgroups of the K tiles.
//
// The general form's decomposition: lane = 8 channels of one token row, but the min/max run down the token rows: each lane keeps
// 8 running minima and maxima over its rows, the 256/(d/8) row slots of the workgroup are
// combined through LDS, one thread per channel derives scale, reciprocal and zero point,
// and a second sweep quantizes and packs.  When a lane's share of the tile fits a few
// registers (HOLD rows: up to 13 x 16 B) the rows stay in registers between the sweeps: 256 threads where those hold the tile, otherwise
// 512 or 1024 (tall_threads in oqm_dispatch.h); of still taller tiles
// the second sweep reads the tile again (from the caches: it was read a moment ago), row by row behind one wait each.
// HBM traffic per element: 2 B read + 0.5 B written + 8/G B of
// (scale, zero) pairs.  The order of the grid, us before / after at 28 layers x 4 heads x 50 x 96 bf16: 8 frames 8.6 / 7.6, 32
// 24.8 / 21.0.  Keys from another tensor, second pass / workgroups of their own: 100 x 80, 1 frame 6.1 / 4.1, 8 12.9 / 11.3; in the row
// waves' form, 50 x 128, 1 frame 5.7 / 3.9, 8 11.7 / 9.5, 32 44.3 / 35.1; 196 x 128, 8 frames 47.5 / 35.8.
#include <type_traits>

#include "oqm_append.h"
#include "oqm_dispatch.h"

namespace oqm {
namespace {

constexpr int kUnroll = 2;

constexpr int kKeyRows = 4;  // rows per lane in flight where only the key is made

// What a workgroup makes.
enum Role : uint32_t { kKeyOnly, kTileK, kTileV };

// SEP: the keys are averaged over another tensor.  Turns a block id into its item.
template <bool SEP>
__device__ __forceinline__ Role role_of(const AppendArgs& a, uint32_t& id) {
    uint32_t role = SEP ? kKeyOnly : kTileK;
    if (id >= a.items) id -= a.items, ++role;
    if (SEP && id >= a.items) id -= a.items, ++role;
    return (Role)role;
}

template <typename IN, bool SEP, int HOLD, int BITS, bool MB, int NT>
__global__ void __launch_bounds__(NT) quantize_append_tokens_kernel(const AppendArgs a) {
    constexpr int EB = elem_bytes<IN>::value;
    constexpr uint32_t CW = BITS;  // bytes of packed codes per lane and row (8 channels)
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    const int G = a.tokens, lpr = a.lanes_per_row, d = lpr * 8;
    uint32_t id = blockIdx.x + a.first_block;
    const Role role = role_of<SEP>(a, id);
    const Item t(a, id);
    const uint32_t kv = role == kTileV ? 1u : 0u;
    const Stored<MB> to(a, t, kv);
    const char* src = (SEP && role == kKeyOnly ? a.ksum : kv ? a.v : a.k) + t.input(a);
    const bool do_sum = SEP ? role == kKeyOnly : role == kTileK;

    const int rpp = a.rows_per_pass;
    const int tid = threadIdx.x;
    const int row0 = div_by(tid, lpr, a.inv_lanes_per_row);
    const int slot = tid - row0 * lpr;
    const bool active = row0 < rpp;
    const uint32_t in_row_bytes = a.row_bytes;
    const uint32_t in_lane = (uint32_t)row0 * in_row_bytes + (uint32_t)slot * 8u * EB;
    const uint32_t code_lane = ((uint32_t)row0 * lpr + slot) * CW;

    __shared__ double shared_buf[NT * 8];            // (min, max) per row slot, then key sums
    extern __shared__ f32x2 fin[];                    // [d] (zero point, 1/scale) per channel
    f32x2* mm = reinterpret_cast<f32x2*>(shared_buf);

    double acc[8];
    float mn[8], mx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        acc[i] = 0.0;
        mn[i] = __builtin_inff();
        mx[i] = -__builtin_inff();
    }

    auto write_key = [&] {
        if (active) {
#pragma unroll
            for (int i = 0; i < 8; ++i) shared_buf[row0 * d + i * lpr + slot] = acc[i];
        }
        __syncthreads();
        float* key = t.key(a);
        for (int q = tid; q < d; q += NT) {
            double sum = 0.0;
            for (int r = 0; r < rpp; ++r) sum += shared_buf[r * d + q];
            key[(q % lpr) * 8 + q / lpr] = (float)(sum / (double)G);
        }
    };
    if (SEP && role == kKeyOnly) {  // uniform
        for (int r0 = 0; r0 < G; r0 += kKeyRows * rpp) {
            Raw8<IN> raw[kKeyRows];
#pragma unroll
            for (int u = 0; u < kKeyRows; ++u) {
                zero_raw(raw[u]);
                if (active && r0 + u * rpp + row0 < G) load_raw(src + (in_lane + (uint32_t)(r0 + u * rpp) * in_row_bytes), raw[u]);
            }
#pragma unroll
            for (int u = 0; u < kKeyRows; ++u) {
                float x[8];
                widen(raw[u], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
            }
        }
        return write_key();
    }

    // ---- sweep 1: per-channel min / max (and the key sums) down the token rows
    const int step = kUnroll * rpp;
    constexpr int kHeld = HOLD > 0 ? HOLD : 1;
    Raw8<IN> held[kHeld];
    auto reduce_row = [&](const Raw8<IN>& raw) {
        float x[8];
        widen(raw, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mn[i] = fminf(mn[i], x[i]);
            mx[i] = fmaxf(mx[i], x[i]);
        }
        if (!SEP && do_sum) {
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
        }
    };
    if (HOLD > 0) {
#pragma unroll
        for (int u = 0; u < kHeld; ++u) {
            zero_raw(held[u]);
            if (active && u * rpp + row0 < G) load_raw(src + (in_lane + (uint32_t)(u * rpp) * in_row_bytes), held[u]);
        }
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if (active && u * rpp + row0 < G) reduce_row(held[u]);
    } else {
        for (int r0 = 0; active && r0 + row0 < G; r0 += step) {
            Raw8<IN> raw[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r0 + u * rpp + row0 < G)
                    load_raw(src + (in_lane + (uint32_t)(r0 + u * rpp) * in_row_bytes), raw[u]);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r0 + u * rpp + row0 < G) reduce_row(raw[u]);
        }
    }
    if (active) {
#pragma unroll
        for (int i = 0; i < 8; ++i) mm[row0 * d + i * lpr + slot] = f32x2{mn[i], mx[i]};  // position, not channel
    }
    __syncthreads();
    // ---- one thread per channel: Eq. 9 over the whole token axis.  The LDS arrays are indexed
    // by position q = i * lpr + slot (channel slot * 8 + i), so that the lanes of a wave touch
    // consecutive words instead of words 64 bytes apart (16-way bank conflicts otherwise).
    for (int q = tid; q < d; q += NT) {
        float cmn = mm[q][0], cmx = mm[q][1];
        for (int r = 1; r < rpp; ++r) {
            cmn = fminf(cmn, mm[r * d + q][0]);
            cmx = fmaxf(cmx, mm[r * d + q][1]);
        }
        cmn = cmn + 0.0f;  // never store -0 as a zero point
        float s = div_levels_exact<BITS>(__fsub_rn(cmx, cmn));
        if (!(s >= 1.17549435e-38f)) s = 0.0f;
        meta_pair stored;
        if constexpr (MB) stored = round_pair_bf16(s, cmn);  // the codes follow the rounded pair
        else stored = f32x2{s, cmn};
        const float inv = s >= 1.17549435e-38f ? rcp_scale<BITS>(s) : 0.0f;
        const int c = (q % lpr) * 8 + q / lpr;
        to.meta[c] = stored;
        fin[q] = f32x2{cmn, inv};
    }
    __syncthreads();

    // ---- sweep 2: quantize and pack
    if (active) {
        float zm[8], zi[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x2 v = fin[i * lpr + slot];
            zm[i] = v[0];
            zi[i] = v[1];
        }
        auto quantize_row = [&](const Raw8<IN>& raw, int rb) {
            float x[8], tq[8];
            widen(raw, x);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                tq[i] = __builtin_fmaf(__fsub_rn(x[i], zm[i]), zi[i], 8388608.0f);
                if constexpr (MB) tq[i] = clamp_code<BITS>(tq[i]);  // m may lie above the minimum
            }
            store_codes8<BITS>(to.codes + (code_lane + (uint32_t)rb * lpr * CW), tq);
        };
        if (HOLD > 0) {
#pragma unroll
            for (int u = 0; u < kHeld; ++u)
                if (u * rpp + row0 < G) quantize_row(held[u], u * rpp);
        } else {
            for (int r0 = 0; r0 + row0 < G; r0 += step) {
                Raw8<IN> raw[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (r0 + u * rpp + row0 < G)
                        load_raw(src + (in_lane + (uint32_t)(r0 + u * rpp) * in_row_bytes), raw[u]);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (r0 + u * rpp + row0 < G) quantize_row(raw[u], r0 + u * rpp);
            }
        }
    }
    if (!do_sum) return;  // uniform per workgroup
    __syncthreads();  // the (min, max) use of shared_buf is over
    write_key();
}

// The form for d = 64, 128, 256 (LPR = d/8 lanes per token row divides a wave).  As few waves as can hold the tile at eight rows per lane (13 where
// that would be more than four waves) own it; a wave reduces its rows with lane swaps, several exchange one (min, max) per channel through LDS behind
// a barrier, one alone needs neither.  Each phase of a launch this short is latency or vector work, not bandwidth: fewer threads per tile mean more
// tiles in flight and fewer of the per-channel steps. The keys are summed while the codes are packed, from the same widened rows and behind the
// exchange that the codes wait for. A key taken from another tensor has workgroups of its own, which hold that tensor's tile. Grid: those, then all K
// tiles, then all V tiles, so that one dense stream of addresses is read at a time and the longer workgroups start first.  Measured, us: 28 layers x
// 4 heads x 50 x 128 (two waves of seven rows), K and V of a layer in turn with the sums in front of the exchange / in turn / V first / K first: 8
// FP16 frames 9.2 / 9.3 / 8.8 / 8.6, 32 bf16 frames (124 MB) 25.6 / 25.9 / 25.3 / 24.3 (5.1 TB/s), 16 13.5 / 13.2 / 12.9 / 12.0; 196 tokens x 4
// frames 15.2 / 14.0 / 13.3 / 12.9.  It takes 88 registers, five waves per SIMD; forcing fewer spills and loses.  At 32 frames one wave of 13 rows
// takes 29.1 us, three waves of five 28.4, four of four 29.8, skipping the dead rows by a branch per row 27.5 (no v_min3 across rows), where this
// form took 25.9; the 256-thread form below 30.1.
template <typename IN, int LPR, int HOLD, int BITS, bool MB, bool SEP>
__global__ void __launch_bounds__(256) quantize_append_rows_kernel(const AppendArgs a, const int waves) {
    constexpr int EB = elem_bytes<IN>::value;
    constexpr uint32_t CW = BITS;  // bytes of packed codes per lane and row (8 channels)
    constexpr int R = 64 / LPR, D = 8 * LPR, CH = LPR / 8;  // rows and channels of a wave's pass; channels a lane finishes
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    extern __shared__ double lds_sum[];             // [waves][D] key sums, then [waves][D] (min, max)
    f32x2* const lds_mm = reinterpret_cast<f32x2*>(lds_sum + waves * D);
    const int G = a.tokens;
    uint32_t id = blockIdx.x + a.first_block;
    const Role role = role_of<SEP>(a, id);
    const Item t(a, id);
    const uint32_t kv = role == kTileV ? 1u : 0u;
    const Stored<MB> to(a, t, kv);
    const char* src = (SEP && role == kKeyOnly ? a.ksum : kv ? a.v : a.k) + t.input(a);
    const bool do_sum = SEP ? role == kKeyOnly : role == kTileK;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row0 = wave * R + lane / LPR, slot = lane % LPR;
    const int step = waves * R;  // token rows per pass
    const int c0 = slot * 8 + (lane / LPR) * CH;  // first channel this lane finishes

    // pass u covers rows [u * step, (u + 1) * step); rows past G repeat the last one (in the cache already)
    Raw8<IN> held[HOLD];
#pragma unroll
    for (int u = 0; u < HOLD; ++u)
        load_raw(src + ((uint32_t)min(u * step + row0, G - 1) * a.row_bytes + (uint32_t)slot * (8u * EB)), held[u]);

    float zm[8], zi[8];
    if (!SEP || role != kKeyOnly) {  // uniform
        float mn[8], mx[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mn[i] = __builtin_inff();
            mx[i] = -__builtin_inff();
        }
#pragma unroll
        for (int u = 0; u < HOLD; ++u) {
            float x[8];
            widen(held[u], x);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                mn[i] = fminf(mn[i], x[i]);
                mx[i] = fmaxf(mx[i], x[i]);
            }
        }
        reduce_rows<LPR>(mn, [](float p, float q) { return fminf(p, q); });
        reduce_rows<LPR>(mx, [](float p, float q) { return fmaxf(p, q); });
        if (waves > 1) {  // uniform
#pragma unroll
            for (int j = 0; j < CH; ++j) lds_mm[wave * D + c0 + j] = f32x2{mn[j], mx[j]};
            __syncthreads();
            for (int w = 0; w < waves; ++w) {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const f32x2 m = lds_mm[w * D + c0 + j];
                    mn[j] = fminf(mn[j], m[0]);
                    mx[j] = fmaxf(mx[j], m[1]);
                }
            }
        }

        // Eq. 9 over the whole token axis, for this lane's channels; then all 8 of its slot
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            float m = mn[j] + 0.0f;  // never store -0 as a zero point
            float s = div_levels_exact<BITS>(__fsub_rn(mx[j], m));
            if (!(s >= 1.17549435e-38f)) s = 0.0f;
            meta_pair stored;
            if constexpr (MB) stored = round_pair_bf16(s, m);  // the codes follow the rounded pair
            else stored = f32x2{s, m};
            if (wave == 0) to.meta[c0 + j] = stored;
            zm[j] = m;
            zi[j] = s >= 1.17549435e-38f ? rcp_scale<BITS>(s) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < HOLD; ++u) forget_widened(held[u]);
        spread_rows<LPR>(zm);
        spread_rows<LPR>(zi);
    }
    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    auto finish_rows = [&](auto codes, auto sums) {
#pragma unroll
        for (int u = 0; u < HOLD; ++u) {
            const int row = u * step + row0;
            float x[8], tq[8];
            widen(held[u], x);
            if constexpr (decltype(codes)::value) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    tq[i] = __builtin_fmaf(__fsub_rn(x[i], zm[i]), zi[i], 8388608.0f);
                    if constexpr (MB) tq[i] = clamp_code<BITS>(tq[i]);  // m may lie above the minimum
                }
            }
            if (row < G) {
                if constexpr (decltype(codes)::value) store_codes8<BITS>(to.codes + ((uint32_t)row * LPR + slot) * CW, tq);
                if constexpr (decltype(sums)::value) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
                }
            }
        }
    };
    if (!do_sum) return finish_rows(std::true_type{}, std::false_type{});  // uniform
    if (SEP && role == kKeyOnly) finish_rows(std::false_type{}, std::true_type{});
    else finish_rows(std::true_type{}, std::true_type{});
    reduce_rows<LPR>(acc, [](double p, double q) { return p + q; });
    if (waves > 1) {
#pragma unroll
        for (int j = 0; j < CH; ++j) lds_sum[wave * D + c0 + j] = acc[j];
        __syncthreads();
        if (wave != 0) return;
        for (int w = 1; w < waves; ++w) {
#pragma unroll
            for (int j = 0; j < CH; ++j) acc[j] += lds_sum[w * D + c0 + j];
        }
    }
    float* key = t.key(a);
#pragma unroll
    for (int j = 0; j < CH; ++j) key[c0 + j] = (float)(acc[j] / (double)G);
}

int64_t set_items(AppendArgs& a, const QuantArgs& q) {
    const int64_t items = (int64_t)q.n_kv_heads * q.n_layers * q.n_frames;  // the API layer keeps them below 2^30
    a.items = (uint32_t)items;
    return items;
}

// Calls go with the code width, the metadata kind and whether the keys come from another tensor as types.
template <typename GO>
hipError_t with_options(const QuantArgs& q, GO go) {
    auto with_source = [&](auto bits, auto mb) { return q.ksum != q.k ? go(bits, mb, std::true_type{}) : go(bits, mb, std::false_type{}); };
    auto with_meta = [&](auto bits) { return q.meta_bf16 ? with_source(bits, std::true_type{}) : with_source(bits, std::false_type{}); };
    return q.bits == 2 ? with_meta(std::integral_constant<int, 2>{}) : with_meta(std::integral_constant<int, 4>{});
}

template <typename IN, int LPR, int HOLD>
hipError_t launch_rows_h(const QuantArgs& q, int waves, hipStream_t s) {
    const size_t lds = waves > 1 ? (size_t)waves * LPR * 8 * (sizeof(double) + sizeof(f32x2)) : 0;
    AppendArgs a = append_args(q, elem_bytes<IN>::value, (uint32_t)q.head_dim);
    auto go = [&](auto bits, auto mb, auto sep) {
        constexpr int B = decltype(bits)::value;
        constexpr bool M = decltype(mb)::value, S = decltype(sep)::value;
        return launch_blocks(a, (S ? 3 : 2) * set_items(a, q), 64 * waves, [&](dim3 grid, dim3 block) {
            launch(quantize_append_rows_kernel<IN, LPR, HOLD, B, M, S>, grid, block, lds, s, a, waves);
        });
    };
    return with_options(q, go);
}

template <typename IN, int LPR>
hipError_t launch_rows(const QuantArgs& a, int waves, int rows, hipStream_t s) {
    if (rows <= 4) return launch_rows_h<IN, LPR, 4>(a, waves, s);
    if (rows <= 6) return launch_rows_h<IN, LPR, 6>(a, waves, s);
    if (rows == 7) return launch_rows_h<IN, LPR, 7>(a, waves, s);
    if constexpr (sizeof(Raw8<IN>) <= 16) {
        if (rows > kMostRows) return launch_rows_h<IN, LPR, kMostRows16Bit>(a, waves, s);
    }
    return launch_rows_h<IN, LPR, kMostRows>(a, waves, s);
}

template <typename IN, int HOLD, int NT = kBlock>
hipError_t launch_h(const QuantArgs& q, hipStream_t s) {
    AppendArgs a = append_args(q, elem_bytes<IN>::value, (uint32_t)q.head_dim);
    a.rows_per_pass = (int32_t)(NT / a.lanes_per_row);
    const size_t lds = (size_t)q.head_dim * sizeof(f32x2);
    auto go = [&](auto bits, auto mb, auto sep) {
        constexpr int B = decltype(bits)::value;
        constexpr bool M = decltype(mb)::value, S = decltype(sep)::value;
        return launch_blocks(a, (S ? 3 : 2) * set_items(a, q), NT, [&](dim3 grid, dim3 block) {
            launch(quantize_append_tokens_kernel<IN, S, HOLD, B, M, NT>, grid, block, lds, s, a);
        });
    };
    return with_options(q, go);
}

template <typename IN>
hipError_t launch_t(const QuantArgs& a, hipStream_t s) {
    if (a.n_frames == 0 || a.n_layers == 0) return hipSuccess;
    const int lpr = a.head_dim / 8;
    if (const int waves = row_waves(lpr, a.group_tokens, sizeof(Raw8<IN>) <= 16)) {
        const int rows = rows_per_lane(lpr, a.group_tokens, waves);
        if (lpr == 8) return launch_rows<IN, 8>(a, waves, rows, s);
        if (lpr == 16) return launch_rows<IN, 16>(a, waves, rows, s);
        return launch_rows<IN, 32>(a, waves, rows, s);
    }
    constexpr bool is_16_bit = sizeof(Raw8<IN>) <= 16;
    constexpr int kMost = is_16_bit ? kMostHeld16Bit : kMostHeld;
    const int trips = held_rows(lpr, a.group_tokens, kBlock);  // rows per lane
    if (trips <= 4) return launch_h<IN, 4>(a, s);
    if (trips <= 8) return launch_h<IN, 8>(a, s);
    if (trips <= kMost) return launch_h<IN, kMost>(a, s);
    switch (tall_threads(lpr, a.group_tokens, is_16_bit)) {
        case 512: return launch_h<IN, kMost, 512>(a, s);
        case 1024: return held_rows(lpr, a.group_tokens, 1024) <= 8 ? launch_h<IN, 8, 1024>(a, s) : launch_h<IN, kMost, 1024>(a, s);
    }
    return launch_h<IN, 0>(a, s);
}

}  // namespace

hipError_t launch_quantize_append_tokens(const QuantArgs& a, int in_dtype, hipStream_t s) {
    switch (in_dtype) {
        case TOM_F32: return launch_t<In_f32>(a, s);
        case TOM_BF16: return launch_t<In_bf16>(a, s);
        case TOM_F16: return launch_t<In_f16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace oqm
