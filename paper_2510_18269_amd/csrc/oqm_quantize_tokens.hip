// Store step with the quantization axis of the paper's Eq. 9: one (scale, zero) pair per
// head and channel, taken over the G tokens of the frame-group (Sec. 3.4, Eq. 8 and Eq. 9),
// plus nibble packing and the summary key, for one head tile per workgroup.
//
// The general form's decomposition: (grid (head, 2*layer + K|V, frame), lane =
// 8 channels of one token row), but the min/max run down the token rows: each lane keeps
// 8 running minima and maxima over its rows, the 256/(d/8) row slots of the workgroup are
// combined through LDS, one thread per channel derives scale, reciprocal and zero point,
// and a second sweep quantizes and packs.  When a lane's share of the tile fits a few
// registers (HOLD rows: up to 13 x 16 B) the rows stay in registers between the sweeps;
// otherwise the second sweep reads the tile again (from the caches: it was read a moment ago).
// HBM traffic per element: 2 B read + 0.5 B written + 8/G B of
// (scale, zero) pairs.
#include <type_traits>

#include "oqm_common.h"
#include "oqm_device.h"
#include "oqm_dispatch.h"

namespace oqm {
namespace {

constexpr int kUnroll = 2;

template <typename IN, bool SEPARATE_SUMMARY, int HOLD, int BITS, bool MB>
__global__ void __launch_bounds__(kBlock) quantize_append_tokens_kernel(const QuantArgs a) {
    constexpr int EB = elem_bytes<IN>::value;
    constexpr uint32_t CW = BITS;  // bytes of packed codes per lane and row (8 channels)
    const int H = a.n_kv_heads, d = a.head_dim, G = a.group_tokens;
    const int h = blockIdx.x;
    const int kv = blockIdx.y & 1;
    const int li = blockIdx.y >> 1;
    const int f = blockIdx.z;
    const int l = a.layer0 + li;
    const int64_t t = (int64_t)a.first_group + f;

    const int lpr = d >> 3;
    const int rpp = kBlock / lpr;
    const int tid = threadIdx.x;
    const int row0 = tid / lpr;
    const int slot = tid - row0 * lpr;
    const bool active = row0 < rpp;

    const int64_t in_off = f * a.stride_frame + li * a.stride_layer + h * a.stride_head;
    const char* src = static_cast<const char*>(kv ? a.v : a.k) + in_off * EB;
    const int64_t tile = (((int64_t)l * 2 + kv) * a.capacity_groups + t) * H + h;
    char* codes_t = reinterpret_cast<char*>(a.codes + tile * ((int64_t)G * d * BITS / 8));
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    meta_pair* meta_t = reinterpret_cast<meta_pair*>(a.meta) + tile * (int64_t)d;  // [d] (scale, zero)
    const uint32_t in_row_bytes = (uint32_t)a.stride_token * EB;
    const uint32_t in_lane = (uint32_t)row0 * in_row_bytes + (uint32_t)slot * 8u * EB;
    const uint32_t code_lane = ((uint32_t)row0 * lpr + slot) * CW;

    __shared__ double shared_buf[kBlock * 8];        // 16 KB: (min, max) per row slot, then key sums
    extern __shared__ f32x2 fin[];                    // [d] (zero point, 1/scale) per channel
    f32x2* mm = reinterpret_cast<f32x2*>(shared_buf);

    const bool do_sum = (kv == 0);
    double acc[8];
    float mn[8], mx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        acc[i] = 0.0;
        mn[i] = __builtin_inff();
        mx[i] = -__builtin_inff();
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
        if (!SEPARATE_SUMMARY && do_sum) {
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
    for (int q = tid; q < d; q += kBlock) {
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
        meta_t[c] = stored;
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
            store_codes8<BITS>(codes_t + (code_lane + (uint32_t)rb * lpr * CW), tq);
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

    if (SEPARATE_SUMMARY) {
        const char* ssrc = static_cast<const char*>(a.ksum) + in_off * EB;
        for (int row = row0; active && row < G; row += rpp) {
            float x[8];
            load8(ssrc + ((int64_t)row * a.stride_token + slot * 8) * EB, IN{}, x);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
        }
    }
    __syncthreads();  // the (min, max) use of shared_buf is over
    if (active) {
#pragma unroll
        for (int i = 0; i < 8; ++i) shared_buf[row0 * d + i * lpr + slot] = acc[i];
    }
    __syncthreads();
    float* key = a.keys + (((int64_t)l * a.capacity_groups + t) * H + h) * d;
    for (int q = tid; q < d; q += kBlock) {
        double sum = 0.0;
        for (int r = 0; r < rpp; ++r) sum += shared_buf[r * d + q];
        key[(q % lpr) * 8 + q / lpr] = (float)(sum / (double)G);
    }
}

// The form for d = 64, 128, 256 (LPR = d/8 lanes per token row divides a wave).  As few waves as
// can hold the tile at eight rows per lane (13 where that would be more than four waves) own it; a wave reduces its rows with lane swaps, several
// exchange one (min, max) and one key sum per channel through LDS behind a single barrier, one
// alone needs neither.  Each phase of a launch this short is latency or vector work, not
// bandwidth: fewer threads per tile mean more tiles in flight and fewer of the per-channel steps.
// Measured (28 layers x 4 heads x 50 x 128, two waves of seven rows, against the 256-thread
// form below): 8 FP16 frames 9.2 / 9.9 us, 32 bf16 frames 25.9 / 30.1 us = 4.6 TB/s.  At 32 frames one wave of 13 rows takes
// 29.1 us, three waves of five 28.4, four of four 29.8; skipping the dead rows by a branch per row
// 27.5 (no v_min3 across rows), keeping the widened rows for the second sweep 26.6.
template <typename IN, int LPR, int HOLD, int BITS, bool MB>
__global__ void __launch_bounds__(256) quantize_append_rows_kernel(const QuantArgs a, const int waves) {
    constexpr int EB = elem_bytes<IN>::value;
    constexpr uint32_t CW = BITS;  // bytes of packed codes per lane and row (8 channels)
    constexpr int R = 64 / LPR, D = 8 * LPR, CH = LPR / 8;  // rows and channels of a wave's pass; channels a lane finishes
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    extern __shared__ double lds_sum[];             // [waves][D] key sums, then [waves][D] (min, max)
    f32x2* const lds_mm = reinterpret_cast<f32x2*>(lds_sum + waves * D);
    const int H = a.n_kv_heads, G = a.group_tokens;
    const int h = blockIdx.x, kv = blockIdx.y & 1, li = blockIdx.y >> 1, f = blockIdx.z;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row0 = wave * R + lane / LPR, slot = lane % LPR;
    const int step = waves * R;  // token rows per pass
    const int c0 = slot * 8 + (lane / LPR) * CH;  // first channel this lane finishes

    const int64_t in_off = f * a.stride_frame + li * a.stride_layer + h * a.stride_head;
    const char* src = static_cast<const char*>(kv ? a.v : a.k) + in_off * EB;
    const int64_t group = (int64_t)a.first_group + f;
    const int64_t tile = (((int64_t)(a.layer0 + li) * 2 + kv) * a.capacity_groups + group) * H + h;
    char* codes_t = reinterpret_cast<char*>(a.codes) + tile * ((int64_t)G * (D * BITS / 8));
    meta_pair* meta_t = static_cast<meta_pair*>(a.meta) + tile * D;
    const uint32_t in_row_bytes = (uint32_t)a.stride_token * EB;
    const bool do_sum = kv == 0;

    // pass u covers rows [u * step, (u + 1) * step); rows past G repeat the last one (in the cache already)
    Raw8<IN> held[HOLD];
#pragma unroll
    for (int u = 0; u < HOLD; ++u)
        load_raw(src + ((uint32_t)min(u * step + row0, G - 1) * in_row_bytes + (uint32_t)slot * (8u * EB)), held[u]);

    double acc[8];
    float mn[8], mx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        acc[i] = 0.0;
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
    if (do_sum) {
#pragma unroll
        for (int u = 0; u < HOLD; ++u) {
            float x[8];
            widen(held[u], x);
            if (u * step + row0 < G) {
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
            }
        }
    }
    reduce_rows<LPR>(mn, [](float p, float q) { return fminf(p, q); });
    reduce_rows<LPR>(mx, [](float p, float q) { return fmaxf(p, q); });
    if (do_sum) reduce_rows<LPR>(acc, [](double p, double q) { return p + q; });
    if (waves > 1) {  // uniform
#pragma unroll
        for (int j = 0; j < CH; ++j) lds_mm[wave * D + c0 + j] = f32x2{mn[j], mx[j]};
        if (do_sum) {
#pragma unroll
            for (int j = 0; j < CH; ++j) lds_sum[wave * D + c0 + j] = acc[j];
        }
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
    float zm[8], zi[8];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        float m = mn[j] + 0.0f;  // never store -0 as a zero point
        float s = div_levels_exact<BITS>(__fsub_rn(mx[j], m));
        if (!(s >= 1.17549435e-38f)) s = 0.0f;
        meta_pair stored;
        if constexpr (MB) stored = round_pair_bf16(s, m);  // the codes follow the rounded pair
        else stored = f32x2{s, m};
        if (wave == 0) meta_t[c0 + j] = stored;
        zm[j] = m;
        zi[j] = s >= 1.17549435e-38f ? rcp_scale<BITS>(s) : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < HOLD; ++u) forget_widened(held[u]);
    spread_rows<LPR>(zm);
    spread_rows<LPR>(zi);
#pragma unroll
    for (int u = 0; u < HOLD; ++u) {
        float x[8], tq[8];
        widen(held[u], x);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            tq[i] = __builtin_fmaf(__fsub_rn(x[i], zm[i]), zi[i], 8388608.0f);
            if constexpr (MB) tq[i] = clamp_code<BITS>(tq[i]);  // m may lie above the minimum
        }
        const int row = u * step + row0;
        if (row < G) store_codes8<BITS>(codes_t + ((uint32_t)row * LPR + slot) * CW, tq);
    }

    if (!do_sum || wave != 0) return;
    float* key = a.keys + (((int64_t)(a.layer0 + li) * a.capacity_groups + group) * H + h) * D;
    for (int w = 1; w < waves; ++w) {
#pragma unroll
        for (int j = 0; j < CH; ++j) acc[j] += lds_sum[w * D + c0 + j];
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) key[c0 + j] = (float)(acc[j] / (double)G);
}

template <typename IN, int LPR, int HOLD>
hipError_t launch_rows_h(const QuantArgs& a, int waves, hipStream_t s) {
    const dim3 grid(a.n_kv_heads, 2 * a.n_layers, a.n_frames), block(64 * waves);
    const size_t lds = waves > 1 ? (size_t)waves * LPR * 8 * (sizeof(double) + sizeof(f32x2)) : 0;
    auto go = [&](auto bits, auto mb) {
        quantize_append_rows_kernel<IN, LPR, HOLD, decltype(bits)::value, decltype(mb)::value><<<grid, block, lds, s>>>(a, waves);
    };
    using std::integral_constant;
    if (a.bits == 2 && a.meta_bf16) go(integral_constant<int, 2>{}, std::true_type{});
    else if (a.bits == 2) go(integral_constant<int, 2>{}, std::false_type{});
    else if (a.meta_bf16) go(integral_constant<int, 4>{}, std::true_type{});
    else go(integral_constant<int, 4>{}, std::false_type{});
    return hipGetLastError();
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

template <typename IN, int HOLD, int BITS, bool MB>
hipError_t launch_m(const QuantArgs& a, hipStream_t s) {
    const dim3 grid(a.n_kv_heads, 2 * a.n_layers, a.n_frames);
    const size_t lds = (size_t)a.head_dim * sizeof(f32x2);
    if (a.ksum != a.k)
        quantize_append_tokens_kernel<IN, true, HOLD, BITS, MB><<<grid, dim3(kBlock), lds, s>>>(a);
    else
        quantize_append_tokens_kernel<IN, false, HOLD, BITS, MB><<<grid, dim3(kBlock), lds, s>>>(a);
    return hipGetLastError();
}

template <typename IN, int HOLD>
hipError_t launch_h(const QuantArgs& a, hipStream_t s) {
    if (a.meta_bf16) return a.bits == 2 ? launch_m<IN, HOLD, 2, true>(a, s) : launch_m<IN, HOLD, 4, true>(a, s);
    return a.bits == 2 ? launch_m<IN, HOLD, 2, false>(a, s) : launch_m<IN, HOLD, 4, false>(a, s);
}

template <typename IN>
hipError_t launch_t(const QuantArgs& a, hipStream_t s) {
    if (a.n_frames == 0 || a.n_layers == 0) return hipSuccess;
    const int lpr = a.head_dim / 8;
    // a separate summary source is one more pass over another tensor: the general form is as fast there
    if (const int waves = a.ksum == a.k ? row_waves(lpr, a.group_tokens, sizeof(Raw8<IN>) <= 16) : 0) {
        const int rows = rows_per_lane(lpr, a.group_tokens, waves);
        if (lpr == 8) return launch_rows<IN, 8>(a, waves, rows, s);
        if (lpr == 16) return launch_rows<IN, 16>(a, waves, rows, s);
        return launch_rows<IN, 32>(a, waves, rows, s);
    }
    const int rpp = kBlock / lpr;
    const int trips = (a.group_tokens + rpp - 1) / rpp;  // rows per lane
    if (trips <= 4) return launch_h<IN, 4>(a, s);
    if (trips <= 8) return launch_h<IN, 8>(a, s);
    if constexpr (sizeof(Raw8<IN>) <= 16) {  // 13 float32 rows would not fit the register budget
        if (trips <= 13) return launch_h<IN, 13>(a, s);
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
