// Store step of Online Quantized Memory on gfx950: 4-bit (or 2-bit) quantization
// of the frame-group tiles of K and V (paper Sec. 3.4, Eq. 8 and Eq. 9), code
// packing, and the summary key (mean of the un-quantized keys over the G tokens
// of the group).
//
// Work decomposition.  A lane owns 8 consecutive channels of one token row: one
// 128-bit load in, one 32-bit word of packed nibbles out, so every load and
// store instruction of a wave covers one contiguous span (1 KB in, 256 B out).
// A quant-group of gs channels lives in gs/8 adjacent lanes; its min and max are
// all-reduced with DPP lane swaps; the first lane of the group stores its
// (scale, zero) pair (8 bytes).
//
// A tile (one (frame, layer, K|V, head) block of G x d) is cut into equal chunks of at most
// two rows per lane (7 x 28 rows at 196 x 128), and every chunk is a workgroup of 256 threads
// (one row per lane is 40 % slower, three to five rows 5 % slower).  Chunked workgroups stream
// faster than whole tiles because the workgroups in flight then cover one dense, moving
// address window.  The summary key needs the column sums over all G rows, and a
// reduction across workgroups costs more than it saves (float64 atomics or
// written-through partials plus an arrival counter add 10 to 40 % to the kernel), so there are two forms:
//
//   quantize_append_kernel      V in chunks; a K tile is walked by one workgroup, four rows per lane
//                               and trip, which sums its columns on the way.  Bound by HBM.  The
//                               1-D grid holds V chunks, then all K tiles, then the last kTail V chunks: a
//                               walk is long (4 trips at 196 x 128), so without chunks behind them the last
//                               walks leave the chip half empty.  Medium launches thus start with the K tiles.
//                               Tall tiles take workgroups of 1024 threads, which walk four times the rows a trip
//                               (walk_threads in oqm_dispatch.h).
//   quantize_append_cut_kernel  K in chunks as well, and the keys by workgroups of their own that read the
//                               tensor to average.  For keys taken from another tensor (that one is read once
//                               either way), and for launches so small that they are bound by the longest chain of
//                               one workgroup and not by the K tiles that are read twice (cut_append in oqm_dispatch.h).
//
// Measured on MI355X, us per call at 28 layers x 4 heads x 196 x 128, bf16.  1 frame (224 tiles): cut 5.2, walk 6.9,
// one workgroup of 1024 threads per tile 5.9.  Walk by frames, K tiles in front of the last kTail chunks / all V chunks
// first / the same with two rows per lane and trip: 4 frames 10.8 / 13.2 / 13.9, 8 23.2 / 27 / 26.5, 16 46.4 / 48.0 / 49.0, 32 (474 MB)
// 90.3 / 90.2 / 91.8 (5.25 TB/s; K cut too, with no key, 86; an arithmetic-free linear stream
// of the byte mix 80).  kTail of 2048 / 3136 / 4096 / 6272 / 10000 at 8 frames: 25.9 / 24.2 / 23.1 / 22.7 / 22.9; at 32
// 90.6 / 89.6 / 89.5 / 89.8 / 90.0.  At 32 frames 512 threads x 4 rows 91.6, 256 x 7 rows 94, a whole tile in
// flight in 512 or 1024 threads 102 / 111; the sums themselves cost nothing; loads without a branch (rows past the end
// read the last one again) 91.6 and 10.7 instead of 9.7 at 3 frames.  Keys from another tensor, one workgroup per K tile
// before / cut: 1 frame 12.8 / 5.2, 8 39 / 34, 32 129.9 / 124 us.  Tall tiles, 28 layers x 4 heads, in a graph, 1024 threads / 256 / cut: 2000 x 128,
// 2 frames 47.4 / 88.3 / 68.7, 6 174 / 225 / 249; 500 x 128, 3 frames 19.6 / 20.7 / 24.3, 32 223 / 232 / 313; 196 x 256 float32, 1 frame
// 9.5 / 12.7 / 12.6.  Chunks of four rows a lane instead of two: 0 to 6 % slower.
//
// The kernel moves 2.64 B per element (bf16 in, gs 64).  At HBM speed that leaves
// room for only about a dozen instructions per element on the plain fp32 vector
// pipe (64 lanes per CU and clock), so the arithmetic is arranged to need few:
//   widen 1, min/max 1, subtract 1, fused scale-and-round 1, pack 1, plus two
//   float64 instructions per element of K for the summary key,
// and the register footprint is kept small: measured, more resident waves help
// this kernel more than deeper software prefetch does.
#include <type_traits>

#include "oqm_append.h"
#include "oqm_dispatch.h"

namespace oqm {
namespace {

constexpr int kChunkRows = 2;  // rows per lane of a chunk
constexpr int kWalkRows = 4;   // rows per lane and trip of a walk
constexpr int kKeyRows = 4;     // rows per lane in flight where columns are summed (seven: 2 to 4 % slower above 400 tiles, 4 % faster at 224)
constexpr int kTail = 6272;    // chunks behind the workgroups that walk a tile: three rounds of the chip

// Where a lane's rows lie within a tile whose rows go `rpp` to a pass of the workgroup.  32-bit byte offsets
// (checked on the host) keep the address arithmetic per row to one add.
template <typename IN, int LPG, int BITS>
struct Lane {
    uint32_t in, in_row, code, code_row;  // offset of the lane's first row, distance of two token rows
    int meta, meta_row;                   // the same in (scale, zero) pairs
    int row0, wave_row0, rpp, slot;       // first row of the lane and of its wave, rows per pass, place within the row
    bool active, meta_writer;
    __device__ __forceinline__ Lane(const AppendArgs& a, int tid) {
        const int lpr = a.lanes_per_row;  // d / 8
        rpp = a.rows_per_pass;
        row0 = div_by(tid, lpr, a.inv_lanes_per_row);
        slot = tid - row0 * lpr;
        active = row0 < rpp;
        wave_row0 = __builtin_amdgcn_readfirstlane(row0);
        in_row = a.row_bytes;
        in = (uint32_t)row0 * in_row + (uint32_t)slot * (8u * elem_bytes<IN>::value);
        code_row = (uint32_t)(lpr * BITS);  // BITS bytes of codes per lane and row
        code = (uint32_t)row0 * code_row + (uint32_t)(slot * BITS);
        meta_row = (uint32_t)lpr / LPG;  // quant-groups per token row
        meta = row0 * meta_row + (uint32_t)slot / LPG;
        meta_writer = (slot & (LPG - 1)) == 0;
    }
};

// Rows r0 + u * rpp of the lane, u < U, as far as they lie before row_end; zeros otherwise.
template <int U, typename IN, typename LANE>
__device__ __forceinline__ void fetch_rows(const char* src, const LANE& n, int r0, int row_end, Raw8<IN> (&buf)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        zero_raw(buf[u]);
        const int rb = r0 + u * n.rpp;
        if (n.active && rb + n.row0 < row_end) load_raw(src + (n.in + (uint32_t)rb * n.in_row), buf[u]);
    }
}

// Quantizes and stores rows that fetch_rows has fetched; with SUM adds them to the lane's column sums.
template <bool SUM, int BITS, bool MB, int LPG, int U, typename IN>
__device__ __forceinline__ void quantize_rows(const Stored<MB>& to, const Raw8<IN> (&buf)[U], const Lane<IN, LPG, BITS>& n, int r0,
                                              int row_end, double (&acc)[8]) {
    typedef typename MetaPair<MB>::type meta_pair;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int rb = r0 + u * n.rpp;
        if (rb + n.wave_row0 >= row_end) break;  // nothing left for this wave (uniform)
        float x[8];
        widen(buf[u], x);
        // Eq. 9: m = min, s = (max - min) / 15 over the quant-group.  All lanes of a
        // quant-group share one row, so a live lane only ever swaps with live lanes.
        float mn = x[0], mx = x[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            mn = fminf(mn, x[i]);
            mx = fmaxf(mx, x[i]);
        }
        group_minmax<LPG>(mn, mx);
        mn = mn + 0.0f;  // never store -0 as a zero point
        float s = div_levels_exact<BITS>(__fsub_rn(mx, mn));
        if (!(s >= 1.17549435e-38f)) s = 0.0f;  // flat or sub-normal range: all codes 0
        meta_pair stored;
        if constexpr (MB) stored = round_pair_bf16(s, mn);  // the codes follow the rounded pair
        const float inv = s >= 1.17549435e-38f ? rcp_scale<BITS>(s) : 0.0f;
        if constexpr (!MB) stored = f32x2{s, mn};
        float tq[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            tq[i] = __builtin_fmaf(__fsub_rn(x[i], mn), inv, 8388608.0f);
            if constexpr (MB) tq[i] = clamp_code<BITS>(tq[i]);  // m may lie above the minimum
        }
        if (n.active && rb + n.row0 < row_end) {
            store_codes8<BITS>(to.codes + (n.code + (uint32_t)rb * n.code_row), tq);
            if (n.meta_writer) to.meta[n.meta + rb * n.meta_row] = stored;
            if constexpr (SUM) {
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
            }
        }
    }
}

// Summary key from the column sums of the lanes: over the rows of a wave by lane swaps (64 / LPR rows of
// LPR lanes each), over the waves in LDS.  One wave's rows hold `8 * LPR` channels, slot * 8 onwards in lane `slot`.
template <int NT, int LPR>
__device__ __forceinline__ void write_key_by_waves(double (&acc)[8], int slot, double* shared, float* key, int G) {
    constexpr int CH = LPR / 8, D = 8 * LPR;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    reduce_rows<LPR>(acc, [](double p, double q) { return p + q; });
#pragma unroll
    for (int j = 0; j < CH; ++j) shared[wave * D + slot * 8 + (lane / LPR) * CH + j] = acc[j];
    __syncthreads();
    if (threadIdx.x < D) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) sum += shared[w * D + threadIdx.x];
        key[threadIdx.x] = (float)(sum / (double)G);
    }
}

template <int NT, typename LANE>
__device__ __forceinline__ void write_key(const AppendArgs& a, const LANE& n, double (&acc)[8], double* shared, float* key) {
    const int lpr = a.lanes_per_row, d = lpr * 8, G = a.tokens;
    if (lpr == 16) return write_key_by_waves<NT, 16>(acc, n.slot, shared, key, G);  // uniform, like the next two
    if (lpr == 8) return write_key_by_waves<NT, 8>(acc, n.slot, shared, key, G);
    if (lpr == 32) return write_key_by_waves<NT, 32>(acc, n.slot, shared, key, G);
    if (n.active) {
#pragma unroll
        for (int i = 0; i < 8; ++i) shared[n.row0 * d + i * lpr + n.slot] = acc[i];
    }
    __syncthreads();
    // position q = i * lpr + slot holds channel slot * 8 + i: the lanes of a wave write
    // consecutive doubles (channel order would put them 64 bytes apart: 16-way bank conflicts)
    for (int q = threadIdx.x; q < d; q += NT) {
        double sum = 0.0;
        for (int r = 0; r < n.rpp; ++r) sum += shared[r * d + q];
        key[(q % lpr) * 8 + q / lpr] = (float)(sum / (double)G);
    }
}

template <typename IN, int LPG, int BITS, bool MB, int NT>
__global__ void __launch_bounds__(NT) quantize_append_kernel(const AppendArgs a) {
    __shared__ double shared[NT * 8];  // key reduction
    request(a);
    const int chunks = a.items * a.chunks, first_walk = max(0, chunks - kTail);
    // One address computation for both roles: a short launch waits for every line of code it has not run before.
    int id = blockIdx.x, row_begin = 0, row_end = a.tokens;
    const bool walk = id >= first_walk && id < first_walk + (int)a.items;
    if (walk) {
        id -= first_walk;
    } else {
        if (id >= first_walk) id -= a.items;
        const int item = div_by(id, a.chunks, a.inv_chunks);
        row_begin = (id - item * a.chunks) * a.chunk_rows;
        row_end = min(row_end, row_begin + a.chunk_rows);
        id = item;
    }
    const Item t(a, id);
    const Stored<MB> to(a, t, walk ? 0u : 1u);
    const char* src = (walk ? a.k : a.v) + t.input(a);
    const Lane<IN, LPG, BITS> n(a, threadIdx.x);
    double acc[8];
    if (!walk) {
        Raw8<IN> buf[kChunkRows];
        fetch_rows(src, n, row_begin, row_end, buf);
        quantize_rows<false>(to, buf, n, row_begin, row_end, acc);
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    for (int r0 = 0; r0 + n.wave_row0 < a.tokens; r0 += kWalkRows * n.rpp) {
        Raw8<IN> buf[kWalkRows];
        fetch_rows(src, n, r0, a.tokens, buf);
        quantize_rows<true>(to, buf, n, r0, a.tokens, acc);
    }
    write_key<NT>(a, n, acc, shared, t.key(a));
}

// Grid: chunks of all K tiles, then of all V tiles, and in front of the last kTail of them the workgroups that
// make the keys, key_parts per K tile of 64 channels each, or one.
template <typename IN, int LPG, int BITS, bool MB>
__global__ void __launch_bounds__(kBlock) quantize_append_cut_kernel(const AppendArgs a) {
    __shared__ double shared[kBlock * 8];  // key reduction
    request(a);
    const uint32_t key_blocks = a.items * a.key_parts, first_key = (uint32_t)max(0, (int)(2u * a.items * (uint32_t)a.chunks) - kTail);
    int id = (int)(blockIdx.x + a.first_block);  // compared as unsigned, but a signed quotient stays in the scalar unit
    Lane<IN, LPG, BITS> n(a, threadIdx.x);
    if ((uint32_t)id < first_key || (uint32_t)id >= first_key + key_blocks) {
        if ((uint32_t)id >= first_key) id -= (int)key_blocks;
        const uint32_t tile = div_by(id, a.chunks, a.inv_chunks), kv = tile < a.items ? 0u : 1u;
        const Item t(a, tile - kv * a.items);
        const Stored<MB> to(a, t, kv);
        const int row_begin = (id - (int)tile * a.chunks) * a.chunk_rows, row_end = min(a.tokens, row_begin + a.chunk_rows);
        Raw8<IN> buf[kChunkRows];
        double unused[8];
        fetch_rows((kv ? a.v : a.k) + t.input(a), n, row_begin, row_end, buf);
        quantize_rows<false>(to, buf, n, row_begin, row_end, unused);
        return;
    }
    id -= first_key;
    const uint32_t item = div_by(id, a.key_parts, a.inv_key_parts), part = id - item * a.key_parts;
    const Item t(a, item);
    const char* src = a.ksum + t.input(a);
    if (a.key_parts > 1) {  // eight lanes per row
        n.rpp = kBlock / 8;
        n.row0 = threadIdx.x >> 3;
        n.slot = threadIdx.x & 7;
        n.active = true;
        n.wave_row0 = __builtin_amdgcn_readfirstlane(n.row0);
        n.in = (uint32_t)n.row0 * n.in_row + (part * 64 + n.slot * 8) * (uint32_t)elem_bytes<IN>::value;
    }
    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    for (int r0 = 0; r0 + n.wave_row0 < a.tokens; r0 += kKeyRows * n.rpp) {
        Raw8<IN> buf[kKeyRows];
        fetch_rows(src, n, r0, a.tokens, buf);
#pragma unroll
        for (int u = 0; u < kKeyRows; ++u) {
            float x[8];
            widen(buf[u], x);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
        }
    }
    if (a.key_parts > 1) write_key_by_waves<kBlock, 8>(acc, n.slot, shared, t.key(a) + part * 64, a.tokens);
    else write_key<kBlock>(a, n, acc, shared, t.key(a));
}

template <typename IN, int LPG, int BITS, bool MB>
hipError_t launch_b(const QuantArgs& q, hipStream_t s) {
    const int64_t items = (int64_t)q.n_kv_heads * q.n_layers * q.n_frames;
    AppendArgs a = append_args(q, elem_bytes<IN>::value, (uint32_t)q.group_tokens * (uint32_t)(q.head_dim / q.qgroup));
    constexpr bool is_16_bit = sizeof(Raw8<IN>) <= 16;
    auto set_chunks = [&](int threads) {
        a.rows_per_pass = (int32_t)((uint32_t)threads / a.lanes_per_row);
        a.chunks = (a.tokens + kChunkRows * a.rows_per_pass - 1) / (kChunkRows * a.rows_per_pass);
        a.chunk_rows = (a.tokens + a.chunks - 1) / a.chunks;  // equal chunks
        a.inv_chunks = reciprocal_u32((uint32_t)a.chunks);
    };
    a.items = (uint32_t)items;
    if (!cut_append(q, is_16_bit)) {
        const int threads = walk_threads(q, is_16_bit);
        set_chunks(threads);
        // One grid.  (The place of this launch within a split one would cost the small launches 1 to 2 %: another argument in front of all
        // addresses.  More workgroups than a grid takes are cut instead.)
        if (items * (a.chunks + 1) < (1LL << 32) / threads) {
            const dim3 grid((unsigned)(items * (a.chunks + 1))), block(threads);
            if (threads == kBlock) launch(quantize_append_kernel<IN, LPG, BITS, MB, kBlock>, grid, block, 0, s, a);
            else launch(quantize_append_kernel<IN, LPG, BITS, MB, kTallBlock>, grid, block, 0, s, a);
            return hipGetLastError();
        }
    }
    set_chunks(kBlock);
    // A chunk has two rows at least and the API layer keeps items * (tokens + 1) below 2^31: 2 * items * chunks fits a signed integer,
    // the ids an unsigned one.
    a.key_parts = (uint32_t)key_parts(q);
    a.inv_key_parts = reciprocal_u32(a.key_parts);
    return launch_blocks(a, items * (2 * a.chunks + (int)a.key_parts), kBlock, [&](dim3 grid, dim3 block) {
        launch(quantize_append_cut_kernel<IN, LPG, BITS, MB>, grid, block, 0, s, a);
    });
}

template <typename IN, int LPG>
hipError_t launch_t(const QuantArgs& a, hipStream_t s) {
    if (a.n_frames == 0 || a.n_layers == 0) return hipSuccess;
    if (a.meta_bf16) return a.bits == 2 ? launch_b<IN, LPG, 2, true>(a, s) : launch_b<IN, LPG, 4, true>(a, s);
    return a.bits == 2 ? launch_b<IN, LPG, 2, false>(a, s) : launch_b<IN, LPG, 4, false>(a, s);
}

template <typename IN>
hipError_t launch_lpg(const QuantArgs& a, hipStream_t s) {
    switch (a.qgroup) {
        case 8: return launch_t<IN, 1>(a, s);
        case 16: return launch_t<IN, 2>(a, s);
        case 32: return launch_t<IN, 4>(a, s);
        case 64: return launch_t<IN, 8>(a, s);
        case 128: return launch_t<IN, 16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_quantize_append(const QuantArgs& a, int in_dtype, hipStream_t s) {
    if (a.qaxis == TOM_QAXIS_TOKENS) return launch_quantize_append_tokens(a, in_dtype, s);
    switch (in_dtype) {
        case TOM_F32: return launch_lpg<In_f32>(a, s);
        case TOM_BF16: return launch_lpg<In_bf16>(a, s);
        case TOM_F16: return launch_lpg<In_f16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace oqm
