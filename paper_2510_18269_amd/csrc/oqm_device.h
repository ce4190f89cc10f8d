// Device-side helpers for the gfx950 kernels: wave64 cross-lane reductions,
// 128-bit loads/stores of packed elements, dtype widening / narrowing.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace oqm {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct In_f32 {};
struct In_bf16 {};
struct In_f16 {};

// n / d for n < 2^32 and a run-time constant d >= 1 whose m = floor(2^32 / d) (2^32 - 1 for
// d == 1) came from the host: the high product is the quotient or one less.
__device__ __forceinline__ uint32_t div_by(uint32_t n, uint32_t d, uint32_t m) {
    const uint32_t q = __umulhi(n, m);
    return n - q * d >= d ? q + 1u : q;
}

// ---- DPP lane exchange ----------------------------------------------------
// dpp_ctrl encodings: quad_perm[1,0,3,2] = 0xB1 (lane ^ 1), quad_perm[2,3,0,1] = 0x4E
// (lane ^ 2), row_half_mirror = 0x141 (lane -> 7 - lane within 8), row_mirror = 0x140
// (lane -> 15 - lane within 16).  After the first two steps all four lanes of a quad hold
// the quad's result, so the mirrors combine whole quads / whole half-rows.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// All-reduce (min and max at once) over aligned sets of LANES lanes, LANES in {1,2,4,8,16}.
template <int LANES>
__device__ __forceinline__ void group_minmax(float& mn, float& mx) {
    if constexpr (LANES >= 2) {
        mn = fminf(mn, dpp_f32<0xB1>(mn));
        mx = fmaxf(mx, dpp_f32<0xB1>(mx));
    }
    if constexpr (LANES >= 4) {
        mn = fminf(mn, dpp_f32<0x4E>(mn));
        mx = fmaxf(mx, dpp_f32<0x4E>(mx));
    }
    if constexpr (LANES >= 8) {
        mn = fminf(mn, dpp_f32<0x141>(mn));
        mx = fmaxf(mx, dpp_f32<0x141>(mx));
    }
    if constexpr (LANES >= 16) {
        mn = fminf(mn, dpp_f32<0x140>(mn));
        mx = fmaxf(mx, dpp_f32<0x140>(mx));
    }
}

// ---- reduction across the token rows of a wave ------------------------------
// A wave holds 64 / LPR token rows of LPR lanes, 8 channels per lane.  reduce_rows combines v[0 .. 8)
// over the rows and leaves each lane with LPR / 8 finished channels: v[j] is then channel
// row * (LPR / 8) + j of the lane's 8.  spread_rows is the way back: every lane gets all 8.  A
// permlane swap serves two channels at once (v_permlane32_swap exchanges the upper half of the first register with
// the lower half of the second, v_permlane16_swap the odd rows of 16 lanes with the even ones),
// so 8 channels take 4 + 2 (+ 1) exchanges and no LDS.
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
// lanes with bit 3 clear end with their a and that of lane + 8, the others with their b and that of lane - 8
__device__ __forceinline__ void swap8(uint32_t& a, uint32_t& b) {
    const bool upper = (__lane_id() & 8u) != 0;
    const uint32_t other = dpp_u32<0x128>(upper ? a : b);  // row_ror:8 = lane ^ 8
    const uint32_t keep = upper ? b : a;
    a = upper ? other : keep;
    b = upper ? keep : other;
}
template <int N>
__device__ __forceinline__ void swap_lanes(uint32_t& a, uint32_t& b) {
    if constexpr (N == 32) swap32(a, b);
    else if constexpr (N == 16) swap16(a, b);
    else swap8(a, b);
}
template <int N>
__device__ __forceinline__ void swap_lanes(float& a, float& b) {
    uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    swap_lanes<N>(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int N>
__device__ __forceinline__ void swap_lanes(double& a, double& b) {
    uint32_t al = (uint32_t)__double2loint(a), ah = (uint32_t)__double2hiint(a);
    uint32_t bl = (uint32_t)__double2loint(b), bh = (uint32_t)__double2hiint(b);
    swap_lanes<N>(al, bl);
    swap_lanes<N>(ah, bh);
    a = __hiloint2double((int)ah, (int)al);
    b = __hiloint2double((int)bh, (int)bl);
}
template <int LPR, typename T, typename OP>
__device__ __forceinline__ void reduce_rows(T (&v)[8], OP op) {
    static_assert(LPR == 8 || LPR == 16 || LPR == 32, "lanes per token row");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        swap_lanes<32>(v[i], v[i + 4]);
        v[i] = op(v[i], v[i + 4]);
    }
    if constexpr (LPR <= 16) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            swap_lanes<16>(v[i], v[i + 2]);
            v[i] = op(v[i], v[i + 2]);
        }
    }
    if constexpr (LPR <= 8) {
        swap_lanes<8>(v[0], v[1]);
        v[0] = op(v[0], v[1]);
    }
}
template <int LPR>
__device__ __forceinline__ void spread_rows(float (&v)[8]) {
    if constexpr (LPR <= 8) {
        v[1] = v[0];
        swap_lanes<8>(v[0], v[1]);
    }
    if constexpr (LPR <= 16) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            v[i + 2] = v[i];
            swap_lanes<16>(v[i], v[i + 2]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i + 4] = v[i];
        swap_lanes<32>(v[i], v[i + 4]);
    }
}

// ---- raw (not yet widened) 8-element loads: p must be 16-byte aligned; widening bf16 / f16 to float32 is exact ----
template <typename T> struct Raw8;
template <> struct Raw8<In_bf16> { u32x4 a; };
template <> struct Raw8<In_f16> { f16x8 a; };
template <> struct Raw8<In_f32> { f32x4 a, b; };

__device__ __forceinline__ void load_raw(const void* p, Raw8<In_bf16>& r) {
    r.a = *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ void load_raw(const void* p, Raw8<In_f16>& r) {
    r.a = *reinterpret_cast<const f16x8*>(p);
}
__device__ __forceinline__ void load_raw(const void* p, Raw8<In_f32>& r) {
    r.a = reinterpret_cast<const f32x4*>(p)[0];
    r.b = reinterpret_cast<const f32x4*>(p)[1];
}
__device__ __forceinline__ void zero_raw(Raw8<In_bf16>& r) { r.a = u32x4{0u, 0u, 0u, 0u}; }
__device__ __forceinline__ void zero_raw(Raw8<In_f16>& r) {
#pragma unroll
    for (int i = 0; i < 8; ++i) r.a[i] = (_Float16)0.0f;
}
__device__ __forceinline__ void zero_raw(Raw8<In_f32>& r) {
    r.a = f32x4{0.f, 0.f, 0.f, 0.f};
    r.b = r.a;
}
// Makes the compiler widen a held row again later instead of keeping the widened copy as well.
__device__ __forceinline__ void forget_widened(Raw8<In_bf16>& r) { asm volatile("" : "+v"(r.a)); }
__device__ __forceinline__ void forget_widened(Raw8<In_f16>& r) { asm volatile("" : "+v"(r.a)); }
__device__ __forceinline__ void forget_widened(Raw8<In_f32>&) {}
__device__ __forceinline__ void widen(const Raw8<In_bf16>& r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(r.a[i] << 16);
        x[2 * i + 1] = __uint_as_float(r.a[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void widen(const Raw8<In_f16>& r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (float)r.a[i];
}
__device__ __forceinline__ void widen(const Raw8<In_f32>& r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = r.a[i];
        x[4 + i] = r.b[i];
    }
}

// ---- correctly rounded float32 a / 15 and 1 / s in three instructions each ----
// One FMA-residual correction step on top of a multiply by the rounded constant 1/15
// (resp. on top of v_rcp_f32).  The repository's division self-check program compares
// both against IEEE division for every input the quantizer can produce (all 2^31
// non-negative finite `a`; every normal `s` up to FLT_MAX / 15) on the GPU: no mismatch.
__device__ __forceinline__ float div15_exact(float a) {
    const float c = 1.0f / 15.0f;
    const float q = __fmul_rn(a, c);
    const float e = __builtin_fmaf(-15.0f, q, a);
    return __builtin_fmaf(e, c, q);
}
// a / 3 (2-bit codes have 3 steps) by the same construction; checked the same way.
__device__ __forceinline__ float div3_exact(float a) {
    const float c = 1.0f / 3.0f;
    const float q = __fmul_rn(a, c);
    const float e = __builtin_fmaf(-3.0f, q, a);
    return __builtin_fmaf(e, c, q);
}
// (max - min) / (2^BITS - 1)
template <int BITS>
__device__ __forceinline__ float div_levels_exact(float a) {
    if constexpr (BITS == 4) return div15_exact(a);
    else return div3_exact(a);
}
__device__ __forceinline__ float rcp_exact(float s) {
    const float r = __builtin_amdgcn_rcpf(s);
    const float e = __builtin_fmaf(-s, r, 1.0f);
    return __builtin_fmaf(e, r, r);
}

// t[i] = fma(x_i - m, 1/s, 2^23): the exact product is rounded once, to an integer,
// ties to even, and that integer sits in the low mantissa bits:
// bits(t) = 0x4B000000 | code.  Packs 8 codes, even channel in the low nibble.
__device__ __forceinline__ uint32_t pack8(const float (&t)[8]) {
    uint32_t m[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = __float_as_uint(t[i]);
    // byte 0 of (m[2j+1] << 4 | m[2j]) is packed byte j; bits 8..23 of it are zero
    const uint32_t b01 = (m[1] << 4) | m[0];
    const uint32_t b23 = (m[3] << 4) | m[2];
    const uint32_t b45 = (m[5] << 4) | m[4];
    const uint32_t b67 = (m[7] << 4) | m[6];
    const uint32_t lo = (b23 << 8) | b01;  // bytes 0, 1 valid
    const uint32_t hi = (b67 << 8) | b45;
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);  // {lo.b0, lo.b1, hi.b0, hi.b1}
}


// 2-bit codes: channel u of the lane's 8 in bits [2u, 2u + 2) of a 16-bit word.  The
// exponent bits 0x4B000000 of every t stay at or above bit 24 under the left shifts.
__device__ __forceinline__ uint32_t pack8_2bit(const float (&t)[8]) {
    uint32_t w = __float_as_uint(t[0]);
#pragma unroll
    for (int i = 1; i < 8; ++i) w |= __float_as_uint(t[i]) << (2 * i);
    return w & 0xffffu;
}

// One lane's 8 codes: a 32-bit word (4-bit codes) or a 16-bit word (2-bit codes).
template <int BITS>
__device__ __forceinline__ void store_codes8(char* p, const float (&t)[8]) {
    if constexpr (BITS == 4) *reinterpret_cast<uint32_t*>(p) = pack8(t);
    else *reinterpret_cast<uint16_t*>(p) = (uint16_t)pack8_2bit(t);
}
// N codes (8, or 4) of BITS bits.  PAST_CACHES: they are not worth a place in the caches.
template <int BITS, int N, bool PAST_CACHES>
__device__ __forceinline__ uint32_t load_codes(const char* p) {
    auto load = [&](auto type) -> uint32_t {
        const auto* q = reinterpret_cast<const decltype(type)*>(p);
        if constexpr (PAST_CACHES) return __builtin_nontemporal_load(q);
        else return *q;
    };
    if constexpr (BITS * N == 32) return load(uint32_t{});
    else if constexpr (BITS * N == 16) return load(uint16_t{});
    else return load(uint8_t{});
}

// 1 / s for a scale of BITS-bit codes.  With 15 steps s <= FLT_MAX / 15 < 2^126 and the
// quotient is always normal; with 3 steps s can exceed 2^126, where the quotient is
// sub-normal and the short sequence does not hold: those (astronomically wide) groups take
// the full IEEE division.
template <int BITS>
__device__ __forceinline__ float rcp_scale(float s) {
    if constexpr (BITS == 2) {
        if (s > 0x1p126f) return __fdiv_rn(1.0f, s);
    }
    return rcp_exact(s);
}

// ---- (scale, zero) pairs as stored: two float32, or two bfloat16 in one 32-bit word -------
template <bool BF16_META> struct MetaPair;
template <> struct MetaPair<false> { typedef f32x2 type; };
template <> struct MetaPair<true> { typedef uint32_t type; };

// Rounds (s, m) to bfloat16 (nearest even, one v_cvt_pk_bf16_f32), returns the stored word
// and replaces s and m by the rounded values, which is what the codes are then taken against.
__device__ __forceinline__ uint32_t round_pair_bf16(float& s, float& m) {
    const f32x2 v = {s, m};
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    s = __uint_as_float(w << 16);
    m = __uint_as_float(w & 0xffff0000u);
    return w;
}
__device__ __forceinline__ f32x2 widen_pair(f32x2 p) { return p; }
__device__ __forceinline__ f32x2 widen_pair(uint32_t w) {
    return f32x2{__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u)};
}
// code + 2^23 clamped to [2^23, 2^23 + levels]: needed once the zero point is no longer the
// exact minimum (bfloat16 metadata); one v_med3_f32
template <int BITS>
__device__ __forceinline__ float clamp_code(float t) {
    return __builtin_amdgcn_fmed3f(t, 8388608.0f, 8388608.0f + (float)((1 << BITS) - 1));
}

template <typename T> struct elem_bytes;
template <> struct elem_bytes<In_f32> { static constexpr int value = 4; };
template <> struct elem_bytes<In_bf16> { static constexpr int value = 2; };
template <> struct elem_bytes<In_f16> { static constexpr int value = 2; };

// ---- storing consecutive float32 values, narrowed round-to-nearest-even ---
__device__ __forceinline__ u32x4 pack_items(In_bf16, const float (&x)[8]) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x2 v = {x[2 * i], x[2 * i + 1]};
        w[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // v_cvt_pk_bf16_f32
    }
    return w;
}

__device__ __forceinline__ u32x4 pack_items(In_f16, const float (&x)[8]) {
    f16x8 h;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // The value must be rounded to float32 first and to binary16 second; the empty asm
        // keeps the compiler from folding a producing FMA and this narrowing into one
        // mixed-precision instruction that rounds only once.
        float v = x[i];
        asm volatile("" : "+v"(v));
        h[i] = (_Float16)v;  // v_cvt_f16_f32, ties to even
    }
    return __builtin_bit_cast(u32x4, h);
}

__device__ __forceinline__ u32x4 pack_items(In_f32, const float (&x)[4]) { return __builtin_bit_cast(u32x4, f32x4{x[0], x[1], x[2], x[3]}); }

template <typename OUT, int N>
__device__ __forceinline__ void store_items(void* p, OUT out, const float (&x)[N]) {
    __builtin_nontemporal_store(pack_items(out, x), reinterpret_cast<u32x4*>(p));
}
// The lanes of a store write every other 16 bytes here, so it must be left to the caches to join the halves of a line.
__device__ __forceinline__ void store_items(void* p, In_f32, const float (&x)[8]) {
    f32x4* o = reinterpret_cast<f32x4*>(p);
    o[0] = f32x4{x[0], x[1], x[2], x[3]};
    o[1] = f32x4{x[4], x[5], x[6], x[7]};
}

}  // namespace oqm
