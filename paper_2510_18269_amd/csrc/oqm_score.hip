// Retrieval scoring on gfx950 (paper Sec. 3.4, Eq. 12; supplement
// "Question-guided single-pass retrieval").
//
//   query_fold_kernel        Q [H_q][T_q][d] -> GQA mean over the r = H_q/H_k consecutive
//                            query heads of a block, then mean over the T_q tokens.
//   score_mean_query_kernel  one dot product (and one key norm) per stored frame-group
//                            against the folded query: a float64 GEMV that streams the
//                            summary keys once; HBM-bound (H_k*d*4 bytes per group).
//   score_fold_query_kernel  both of these in one launch, for short questions.
//   score_token_gemm_kernel  per-token scores [T_q x H_k*d] x [H_k*d x T] on the matrix
//                            cores (v_mfma_f64_16x16x4_f64), then the token mean; small launches
//                            split the contraction over waves (score_token_split_kernel), and
//                            most of these fold the query themselves (score_token_fold_kernel).
//
// Everything accumulates in float64 (the CDNA vector and matrix pipes run it at
// full rate), so the float32 scores handed to top-k agree with a float64
// reference up to the final rounding, and the selected indices with them.
#include <type_traits>

#include "oqm_common.h"
#include "oqm_device.h"
#include "oqm_dispatch.h"

namespace oqm {
namespace {

// Requests the arguments in one go: the compiler would load them where they are used, one round trip through the
// scalar cache after the other.
__device__ __forceinline__ void request(const ScoreArgs& a) {
    asm volatile("" ::"s"(a.keys), "s"(a.q), "s"(a.scores), "s"(a.ws_qbar), "s"(a.ws_qtok), "s"(a.score_stride),
                 "s"(a.n_kv_heads), "s"(a.n_q_heads), "s"(a.head_dim), "s"(a.capacity_groups), "s"(a.layer0), "s"(a.t_q),
                 "s"(a.n_groups), "s"(a.sim));
}

// Sum of a double over an aligned set of 16 lanes (DPP swaps; valid in all 16 lanes).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row16_sum_f64(double v) {
    v += dpp_f64<0xB1>(v);   // lane ^ 1
    v += dpp_f64<0x4E>(v);   // lane ^ 2
    v += dpp_f64<0x141>(v);  // the other quad of the 8
    v += dpp_f64<0x140>(v);  // the other half of the 16
    return v;
}
// ... over aligned sets of 16, 32 or all 64 lanes of a wave (valid in all of them).
template <int LANES>
__device__ __forceinline__ double lanes_sum_f64(double v) {
    v = row16_sum_f64(v);
    if constexpr (LANES >= 32) {
        double w = v;
        swap_lanes<16>(v, w);
        v += w;
    }
    if constexpr (LANES >= 64) {
        double w = v;
        swap_lanes<32>(v, w);
        v += w;
    }
    return v;
}

// Sum of the four lanes of a wave that are equal modulo 16 (valid in all of them).
__device__ __forceinline__ double rows16_sum_f64(double v) {
    double w = v;
    swap_lanes<16>(v, w);
    v += w;
    w = v;
    swap_lanes<32>(v, w);
    return v + w;
}

// A sum over the workgroup: every wave puts its share, the total can be read behind a barrier.
__device__ __forceinline__ void put_wave_sum(double v, double* wsum) {
    v = lanes_sum_f64<64>(v);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
}
template <int WAVES>
__device__ __forceinline__ double total_of(const double* wsum) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) v += wsum[w];
    return v;
}
// |q-bar|^2 of a layer, from what query_fold_kernel has left: the first elements are requested where this is made, and put() behind the work that
// their latency shall not hold up (summed in front of it, 2000 of the 10800 cycles of a split workgroup with one tile of tokens: 28 layers x 100
// groups x 10 tokens 13.8 -> 13.3 us, 17 x 167 x 10 at 5 heads of 256 18.3 -> 17.5, 28 x 1024 x 64 62.9 -> 62.3, with the sums over lanes by swaps).
template <int THREADS>
struct QueryNorm2 {
    const double* qbar;
    int HD;
    double first;
    __device__ __forceinline__ QueryNorm2(const ScoreArgs& a, int li, int HD_) : qbar(a.ws_qbar + (int64_t)li * HD_), HD(HD_) {
        first = qbar[min((int)threadIdx.x, HD - 1)];
    }
    __device__ __forceinline__ void put(double* wsum) const {
        double sq = (int)threadIdx.x < HD ? first * first : 0.0;
        for (int e = threadIdx.x + THREADS; e < HD; e += THREADS) {
            const double qb = qbar[e];
            sq = fma(qb, qb, sq);
        }
        put_wave_sum(sq, wsum);
    }
};

// Column sums over the row slots of a wave where lpr (d/8) lanes per row divide it: one row of d sums per wave in `red`,
// in channel order.  Every lane of the wave takes part.
__host__ __device__ __forceinline__ bool rows_divide_a_wave(int lpr) { return lpr == 8 || lpr == 16 || lpr == 32; }
__device__ __forceinline__ void join_rows_of_wave(double (&acc)[8], int lpr, int slot, double* red) {
    const int lane = threadIdx.x & 63;
    auto join = [&](auto lanes) {
        constexpr int LPR = decltype(lanes)::value, CH = LPR / 8;
        reduce_rows<LPR>(acc, [](double p, double q) { return p + q; });
#pragma unroll
        for (int j = 0; j < CH; ++j) red[(threadIdx.x >> 6) * (8 * LPR) + slot * 8 + (lane / LPR) * CH + j] = acc[j];
    };
    if (lpr == 16) join(std::integral_constant<int, 16>{});  // uniform
    else if (lpr == 8) join(std::integral_constant<int, 8>{});
    else join(std::integral_constant<int, 32>{});
}

// ------------------------------------------------------------------ query fold
// grid (H_k * parts, n_layers); a workgroup owns d / parts channels of a KV head: kFoldThreads threads = row slots x lanes of 8 channels.  The r *
// T_q rows of a KV head are contiguous in Q: the mean alone is one sum over them.  TOKENS: every token's mean over the r heads is wanted too, so a
// slot takes whole tokens.  Bound by latency and by what the few compute units that take part can load, hence parts of 64 channels in small launches
// (fold_parts in oqm_dispatch.h).  28 layers x 28 heads of 128 in a graph of the whole question, 256 threads per head / 512 / 512 per part: 32 tokens
// 5.4 / 4.5 / 4.4 us, 64 7.5 / 5.7 / 5.0, 64 with every token kept 10.2 / 9.4 / 7.0.  Rows that no slot of the workgroup has are not converted (8
// rows a trip, 0.1 us each): mean query of one token over 28 x 1024 groups 21.2 -> 19.6 us, fused with the scores of one layer x 256 groups 8.9 ->
// 8.3, 16 rows 12.1 -> 11.9.  (Not worth its branches in score_token_fold_kernel, where the heads of a turn are few.)
template <typename QT, bool TOKENS>
__global__ void __launch_bounds__(kFoldThreads) query_fold_kernel(const ScoreArgs a, const int parts) {
    constexpr int EB = elem_bytes<QT>::value;
    request(a);
    const int h = blockIdx.x / parts, li = blockIdx.y;
    const int H = a.n_kv_heads, Tq = a.t_q;
    const int r = a.n_q_heads / H;
    const int64_t HD = (int64_t)H * a.head_dim;
    const int d = a.head_dim / parts, c0 = (blockIdx.x - h * parts) * d;  // channels of this workgroup
    const int lpr = d >> 3;
    const int jn = kFoldThreads / lpr;
    const int tid = threadIdx.x;
    const int jl = tid / lpr;
    const int slot = tid - jl * lpr;
    const bool active = jl < jn;
    const uint32_t row_bytes = (uint32_t)a.head_dim * EB;
    const char* q = static_cast<const char*>(a.q) + ((int64_t)li * H + h) * r * Tq * row_bytes + (c0 + slot * 8) * EB;

    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    constexpr int kRows = 8;  // rows of a lane in flight
    if (!TOKENS) {
        const int64_t rows = (int64_t)r * Tq;
        const int trip = kRows * jn;
        for (int64_t base = 0; base < rows; base += trip) {  // uniform
            const char* src = q + base * row_bytes;
            const int left = active ? (int)min(rows - base, (int64_t)trip) : 0;
            Raw8<QT> raw[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                zero_raw(raw[u]);
                const int row = jl + u * jn;
                if (row < left) load_raw(src + (uint32_t)row * row_bytes, raw[u]);
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                if (base + u * jn >= rows) break;  // uniform: nothing but zeros from here on
                float x[8];
                widen(raw[u], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
            }
        }
    }
    if (TOKENS && active) {
        const double inv_r = 1.0 / (double)r;
        for (int j = jl; j < Tq; j += jn) {
            double qt[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) qt[i] = 0.0;
            for (int g0 = 0; g0 < r; g0 += kRows) {
                Raw8<QT> raw[kRows];
#pragma unroll
                for (int g = 0; g < kRows; ++g) {
                    zero_raw(raw[g]);
                    if (g0 + g < r) load_raw(q + ((uint64_t)(g0 + g) * Tq + j) * row_bytes, raw[g]);
                }
#pragma unroll
                for (int g = 0; g < kRows; ++g) {
                    if (g0 + g >= r) break;  // uniform
                    float x[8];
                    widen(raw[g], x);
#pragma unroll
                    for (int i = 0; i < 8; ++i) qt[i] += (double)x[i];
                }
            }
            f64x2* dst = reinterpret_cast<f64x2*>(a.ws_qtok + ((int64_t)li * Tq + j) * HD + (int64_t)h * a.head_dim + c0 + slot * 8);
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                qt[i] = qt[i] * inv_r;
                qt[i + 1] = qt[i + 1] * inv_r;
                dst[i / 2] = f64x2{qt[i], qt[i + 1]};
                acc[i] += qt[i];
                acc[i + 1] += qt[i + 1];
            }
        }
    }
    const double share = 1.0 / (TOKENS ? (double)Tq : (double)r * (double)Tq);
    __shared__ double red[kFoldThreads * 8];
    const bool by_waves = rows_divide_a_wave(lpr);  // uniform
    if (by_waves) {
        join_rows_of_wave(acc, lpr, slot, red);
    } else if (active) {
#pragma unroll
        for (int i = 0; i < 8; ++i) red[jl * d + i * lpr + slot] = acc[i];  // position order: no bank conflicts
    }
    __syncthreads();
    for (int p = tid; p < d; p += kFoldThreads) {  // channel p, or position p = i * lpr + slot, which holds channel slot * 8 + i
        const int n = by_waves ? kFoldThreads / 64 : jn;
        double sum = 0.0;
        for (int j = 0; j < n; ++j) sum += red[j * d + p];
        a.ws_qbar[(int64_t)li * HD + (int64_t)h * a.head_dim + c0 + (by_waves ? p : (p % lpr) * 8 + p / lpr)] = sum * share;
    }
}

// ------------------------------------------------------------------ mean-query GEMV
constexpr int kScoreChunks = 8;  // 16-byte key loads per lane that are in flight together

// q-bar in LDS: the W lanes of a frame-group read consecutive 16-byte pairs, so element e = 4W c + 4s + i (piece c, lane s, i < 4)
// sits at ((2c + i/2) * W + s) * 2 + i%2 (in element order the lanes' pairs would be 32 bytes apart: bank conflicts on every read).
template <int W>
__device__ __forceinline__ int staged_at(int e) {
    const int c = e / (4 * W), sl = (e >> 2) & (W - 1), i = e & 3;
    return (((2 * c + (i >> 1)) * W + sl) << 1) + (i & 1);
}

// Which lanes load: a key of whole trips of CH pieces; of one trip whose last piece is not whole; any other.  What lies past the
// end of the key is zero in the registers and in the staged q-bar.
enum Rest { kNoRest, kLastPiece, kAnyPiece };

// Key of one group, CH pieces of 4W channels at a time.  W lanes work on a group: lane `sub` of them takes floats
// [4W c + 4 sub, 4W c + 4 sub + 4) for c = 0, 1, ..., so every load instruction of the W lanes covers 16W contiguous bytes.
template <int W, int CH, Rest REST>
struct KeyPieces {
    f32x4 x[CH];
    template <bool PAST_CACHES = false>
    __device__ __forceinline__ void load(const float* key, int e0, int HD, int sub) {
        auto piece = [](const float* p) {
            const f32x4* q = reinterpret_cast<const f32x4*>(p);
            if constexpr (PAST_CACHES) return __builtin_nontemporal_load(q);
            else return *q;
        };
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int e = e0 + c * (4 * W) + sub * 4;
            if (REST == kNoRest || (REST == kLastPiece && c < CH - 1)) {
                x[c] = piece(key + e);
            } else {
                x[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (e < HD) x[c] = piece(key + e);
            }
        }
    }
};

// Dot product and norm of one group's key (its first pieces already in `first`) against the staged query, and the score.
// No branch around the products: the LDS reads of all pieces are then in flight together (with one, this function took 3000 of the 10000 cycles that
// a workgroup of score_fold_query_kernel lives, now 1800; 1 layer x 256 groups x 16 tokens 7.7 -> 6.6 us).
template <bool PAST_CACHES, int W, int CH, Rest REST>
__device__ __forceinline__ void score_of_group(const ScoreArgs& a, const double* qbar, const KeyPieces<W, CH, REST>& first, const float* key,
                                               int HD, int sub, int t, int li, double query_norm) {
    double dot = 0.0, nk2 = 0.0;
    constexpr int trip = 4 * W * CH;
    KeyPieces<W, CH, REST> next = first;
    for (int e0 = 0; REST == kLastPiece ? e0 == 0 : e0 < HD; e0 += trip) {
        const KeyPieces<W, CH, REST> cur = next;
        if (REST != kLastPiece && e0 + trip < HD) next.template load<PAST_CACHES>(key, e0 + trip, HD, sub);  // uniform
        const f64x2* q = reinterpret_cast<const f64x2*>(qbar + e0) + sub;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const f64x2 q01 = q[2 * c * W], q23 = q[(2 * c + 1) * W];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double kd = (double)cur.x[c][i];
                dot = fma(i < 2 ? q01[i] : q23[i - 2], kd, dot);
                nk2 = fma(kd, kd, nk2);
            }
        }
    }
    dot = lanes_sum_f64<W>(dot);
    nk2 = lanes_sum_f64<W>(nk2);
    if (sub == 0 && t < a.n_groups) {
        double s = dot;
        if (a.sim == TOM_SIM_COSINE) s = dot / (fmax(query_norm, 1e-12) * fmax(sqrt(nk2), 1e-12));
        a.scores[(int64_t)li * a.score_stride + t] = (float)s;
    }
}

// grid (ceil(T / (256 / W)), n_layers); dynamic LDS: H_k*d doubles (q-bar), padded to whole trips of CH pieces.
template <int W, int CH, Rest REST, bool PAST_CACHES>
__global__ void __launch_bounds__(kBlock) score_mean_query_kernel(const ScoreArgs a) {
    extern __shared__ __align__(16) double qbar[];
    const int li = blockIdx.y;
    const int HD = a.n_kv_heads * a.head_dim;
    const int tid = threadIdx.x, sub = tid & (W - 1);
    const float* keys = a.keys + ((int64_t)(a.layer0 + li) * a.capacity_groups) * HD;
    const int t = blockIdx.x * (kBlock / W) + tid / W;
    const int tc = min(t, a.n_groups - 1);  // the tail re-reads the last group
    const float* key = keys + (int64_t)tc * HD;
    // The first key loads do not depend on the query: issue them before q-bar is staged.
    KeyPieces<W, CH, REST> first;
    first.template load<PAST_CACHES>(key, 0, HD, sub);

    const int padded = REST == kNoRest ? HD : REST == kLastPiece ? 4 * W * CH : (HD + 4 * W * CH - 1) / (4 * W * CH) * (4 * W * CH);
    __shared__ double wsum[kBlock / 64];
    double sq = 0.0;
    for (int e = tid; e < padded; e += kBlock) {
        const double qb = REST == kNoRest || e < HD ? a.ws_qbar[(int64_t)li * HD + e] : 0.0;
        qbar[staged_at<W>(e)] = qb;
        sq = fma(qb, qb, sq);
    }
    put_wave_sum(sq, wsum);
    __syncthreads();
    const double nq = sqrt(total_of<kBlock / 64>(wsum));

    score_of_group<PAST_CACHES>(a, qbar, first, key, HD, sub, t, li, nq);
}

// Fold and score in one launch, for questions short enough that every workgroup can fold the query
// of its layer by itself.  grid (ceil(T / 32), n_layers), 512 threads; dynamic LDS as above.
// The r * T_q rows of a KV head are contiguous in Q, so the mean over heads and tokens is one
// sum over a run of rows: head h gets the same number of row slots (d/8 lanes each) of the
// workgroup.  The key loads are in flight meanwhile.
// Row slots per KV head and the reciprocals for div_by.  Not part of ScoreArgs: the other kernels' arguments then
// stay within two 64-byte lines.
struct FoldSplit {
    uint32_t slots, inv_slots, inv_lanes_per_row, inv_head_dim;
    int32_t waves;  // of a head, where its slots are whole waves and rows divide a wave; or 0
};

template <typename QT, int CH, Rest REST>
__global__ void __launch_bounds__(kFoldThreads) score_fold_query_kernel(const ScoreArgs a, const FoldSplit f) {
    constexpr int EB = elem_bytes<QT>::value;
    constexpr int kRows = 8;  // query rows per lane in flight
    extern __shared__ __align__(16) double qbar[];
    __shared__ double red[kFoldThreads * 8];
    __shared__ double wsum[kFoldThreads / 64];
    request(a);
    const int li = blockIdx.y;
    const int H = a.n_kv_heads, d = a.head_dim, HD = H * d;
    const int tid = threadIdx.x, sub = tid & 15;
    const float* keys = a.keys + ((int64_t)(a.layer0 + li) * a.capacity_groups) * HD;
    const int t = blockIdx.x * (kFoldThreads / 16) + (tid >> 4);
    const int tc = min(t, a.n_groups - 1);  // the tail re-reads the last group
    const float* key = keys + (int64_t)tc * HD;
    KeyPieces<16, CH, REST> first;
    first.load(key, 0, HD, sub);

    const double share = 1.0 / (double)((a.n_q_heads / H) * a.t_q);
    const int lpr = d >> 3;
    const int s = div_by(tid, lpr, f.inv_lanes_per_row), slot = tid - s * lpr;
    const int h = div_by(s, f.slots, f.inv_slots), part = s - h * f.slots;
    if (h < H) {
        const int rows = (a.n_q_heads / H) * a.t_q;  // small: the launcher bounds the query
        const char* q = static_cast<const char*>(a.q) + (((int64_t)li * H + h) * rows * d + slot * 8) * EB;
        double acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.0;
        for (int r0 = 0; r0 < rows; r0 += kRows * (int)f.slots) {  // uniform
            Raw8<QT> raw[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                zero_raw(raw[u]);
                const int row = r0 + u * (int)f.slots + part;
                if (row < rows) load_raw(q + (int64_t)row * d * EB, raw[u]);
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                if (r0 + u * (int)f.slots >= rows) break;  // uniform: nothing but zeros from here on
                float x[8];
                widen(raw[u], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (double)x[i];
            }
        }
        if (f.waves > 0) {
            join_rows_of_wave(acc, lpr, slot, red);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) red[s * d + i * lpr + slot] = acc[i];  // position order: no bank conflicts
        }
    }
    __syncthreads();
    double sq = 0.0;
    const int padded = REST == kNoRest ? HD : REST == kLastPiece ? CH * 64 : (HD + CH * 64 - 1) / (CH * 64) * (CH * 64);
    for (int e = tid; e < padded; e += kFoldThreads) {
        if (REST != kNoRest && e >= HD) {
            qbar[staged_at<16>(e)] = 0.0;
            continue;
        }
        const int hh = div_by(e, d, f.inv_head_dim), p = e - hh * d;
        int at = e;
        double sum = 0.0;
        if (f.waves > 0) {  // channel p of head hh
            for (int w = 0; w < f.waves; ++w) sum += red[(hh * f.waves + w) * d + p];
        } else {  // position p
            for (int w = 0; w < f.slots; ++w) sum += red[(hh * f.slots + w) * d + p];
            const int i8 = div_by(p, lpr, f.inv_lanes_per_row);
            at = hh * d + (p - i8 * lpr) * 8 + i8;
        }
        const double qb = sum * share;
        qbar[staged_at<16>(at)] = qb;
        sq += qb * qb;
    }
    put_wave_sum(sq, wsum);
    __syncthreads();
    score_of_group<false>(a, qbar, first, key, HD, sub, t, li, sqrt(total_of<kFoldThreads / 64>(wsum)));
}

// ------------------------------------------------------------------ per-token GEMM
// S[j][t] = sum_e qtok[j][e] * key[t][e], j < T_q query tokens, t < T groups, e < H_k*d.
// Unit of work = (layer, 64 consecutive groups): one workgroup of 4 waves; wave w owns groups
// n0 + 16w .. + 15 and up to four 16-token row tiles.  With units of 32 groups (gemm_width in oqm_dispatch.h) waves w and w + 2
// own the same groups and half of the row tiles each.  Operands are staged through LDS in
// chunks of kGemmK along e.
//
// Workgroup id -> unit.  Ids go round-robin over the eight XCDs, each with its own L2, so
// XCD x is given the contiguous run of units [x * per, (x + 1) * per): it then touches the
// folded query block (T_q x H_k*d float64, 256 KB at 64 x 512) of about n_layers / 8 + 1
// layers instead of every layer's (with a (tile, layer) grid every XCD fetched every layer's
// block: 118 MB of traffic for 72 MB of operands at 28 layers x 1024 groups).
//
// v_mfma_f64_16x16x4_f64 register layout (checked on hardware by the GPU tests through
// the per-token score output): lane = 16*kk + i supplies A[i][kk] and B[kk][i]; lane
// 16*g + j holds D[4*v + g][j] in accumulator register v.
constexpr int kGemmM = 64;
constexpr int kGemmK = 32;
// Row pitches of the staged operands.  A fragment read takes element (row fi, column kk) per
// lane: with 34 doubles per row the 32 lanes of a half-wave fall on 4*fi + 2*kk, i.e. on all
// 32 even banks once (a pitch of 36 puts rows fi and fi + 8 on the same banks: measured 9 %
// slower); with 36 floats per row the 64 lanes of a B read fall on 64 different banks.
constexpr int kLdA = kGemmK + 2;  // doubles
constexpr int kLdB = kGemmK + 4;  // floats

__device__ __forceinline__ int mfma_d_row(int lane, int v) { return 4 * v + (lane >> 4); }

// One staged chunk: kGemmK/4 MFMA steps for MT row tiles of 16 tokens against the 16 groups
// of this wave.  No branches inside, so the LDS reads of a step are issued together.
template <int MT>
__device__ __forceinline__ void mma_chunk(const double* __restrict__ As, const float* __restrict__ Bs,
                                          f64x4 (&acc)[MT], double& nk2c, int tile, int fi,
                                          int kk) {
#pragma unroll
    for (int ks = 0; ks < kGemmK / 4; ++ks) {
        const double bv = (double)Bs[(tile * 16 + fi) * kLdB + ks * 4 + kk];
        double av[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) av[m] = As[(m * 16 + fi) * kLdA + ks * 4 + kk];
        nk2c = fma(bv, bv, nk2c);
#pragma unroll
        for (int m = 0; m < MT; ++m)
            acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[m], bv, acc[m], 0, 0, 0);
    }
}

// One block of up to 64 query rows against NG group tiles: the chunk loop with the row-tile count fixed at compile
// time, so the accumulators stay in place across the whole contraction.
template <int MT, int NG, int SIZE>
__device__ __forceinline__ void gemm_rows(const ScoreArgs& a, double (&As)[2][SIZE], float (&Bs)[2][NG * 16 * kLdB],
                                          const double* qtok, const float* keys, int m0, int n0, int li,
                                          double& colsum, double& nk2) {
    const int HD = a.n_kv_heads * a.head_dim;
    const int T = a.n_groups, Tq = a.t_q;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fi = lane & 15, kk = lane >> 4;
    constexpr int kParts = 4 / NG, WT = MT / kParts;  // WT: row tiles of a wave
    const int tile = NG == 4 ? wave : wave % NG, part = NG == 4 ? 0 : wave / NG;  // constants where they can be: `part` enters every LDS address (units of 64 are 1 % faster by it)
    const int n_chunks = (HD + kGemmK - 1) / kGemmK;
    constexpr int kALanes = kGemmK / 2, kBLanes = kGemmK / 4;
    constexpr int kAPass = kBlock / kALanes, kBPass = kBlock / kBLanes;
    constexpr int kARows = (MT * 16 + kAPass - 1) / kAPass, kBRows = NG * 16 / kBPass;
    const int a_row = tid / kALanes, a_col = (tid % kALanes) * 2;
    const int b_row = tid / kBLanes, b_col = (tid % kBLanes) * 4;
    const int rows = min(kGemmM, Tq - m0);

    f64x4 acc[WT];
#pragma unroll
    for (int m = 0; m < WT; ++m) acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
    double nk2c = 0.0;
    double ra[kARows][2];
    f32x4 rb[kBRows];
    auto load_chunk = [&](int c) {
        const int k0 = c * kGemmK;
#pragma unroll
        for (int i = 0; i < kARows; ++i) {
            const int rr = a_row + i * kAPass;
            ra[i][0] = 0.0;
            ra[i][1] = 0.0;
            if (rr < rows && k0 + a_col < HD) {
                const double* p = qtok + (int64_t)(m0 + rr) * HD + k0 + a_col;
                ra[i][0] = p[0];
                ra[i][1] = p[1];
            }
        }
#pragma unroll
        for (int i = 0; i < kBRows; ++i) {
            const int rr = b_row + i * kBPass;
            rb[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (n0 + rr < T && k0 + b_col < HD)
                rb[i] = *reinterpret_cast<const f32x4*>(keys + (int64_t)(n0 + rr) * HD + k0 + b_col);
        }
    };
    auto store_chunk = [&](int stage) {
#pragma unroll
        for (int i = 0; i < kARows; ++i) {
            const int rr = a_row + i * kAPass;
            if (rr < MT * 16) {
                As[stage][rr * kLdA + a_col] = ra[i][0];
                As[stage][rr * kLdA + a_col + 1] = ra[i][1];
            }
        }
#pragma unroll
        for (int i = 0; i < kBRows; ++i) {
            const int rr = b_row + i * kBPass;
#pragma unroll
            for (int j = 0; j < 4; ++j) Bs[stage][rr * kLdB + b_col + j] = rb[i][j];
        }
    };

    __syncthreads();  // the previous row block no longer reads LDS
    load_chunk(0);
    store_chunk(0);
    __syncthreads();
    for (int c = 0; c < n_chunks; ++c) {
        const int stage = c & 1;
        if (c + 1 < n_chunks) load_chunk(c + 1);  // in flight during the MFMAs below
        mma_chunk<WT>(As[stage] + part * WT * 16 * kLdA, Bs[stage], acc, nk2c, tile, fi, kk);
        if (c + 1 < n_chunks) store_chunk(stage ^ 1);  // that stage was consumed before the last barrier
        __syncthreads();
    }
    if (m0 == 0) nk2 = nk2c;
    const int t = n0 + tile * 16 + fi;
#pragma unroll
    for (int m = 0; m < WT; ++m) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = m0 + (part * WT + m) * 16 + mfma_d_row(lane, v);
            colsum += acc[m][v];  // rows >= T_q were staged as zeros
            if (a.token_scores && j < Tq && t < T)
                a.token_scores[((int64_t)li * Tq + j) * T + t] = (float)acc[m][v];
        }
    }
}

// MOST: row tiles of a pass.  With one or two the whole question is one pass, and with registers and LDS for them alone six or four workgroups share
// a compute unit instead of three: 28 layers x 2200 groups x 2 heads of 128 x 16 tokens 29.3 -> 26.5 us (whole question, k = 1), 32 tokens 37.9 ->
// 35.3, 2000 x 1 head of 64 x 16 18.5 -> 16.6; up to one round of the chip 1 to 2 %.  Three tiles gain nothing.
template <int MOST, int NG>
__global__ void __launch_bounds__(kBlock) score_token_gemm_kernel(const ScoreArgs a) {
    // two LDS stages: chunk c is multiplied while chunk c+1 travels global -> registers -> LDS
    __shared__ double As[2][MOST * 16 * kLdA];
    __shared__ float Bs[2][NG * 16 * kLdB];
    const int unit = (int)(blockIdx.x & 7u) * a.gemm_units_per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= a.gemm_units) return;  // uniform per workgroup
    const int li = div_by(unit, a.gemm_tiles_per_layer, a.inv_gemm_tiles_per_layer);
    const int n0 = (unit - li * a.gemm_tiles_per_layer) * (NG * 16);
    const int HD = a.n_kv_heads * a.head_dim;
    const int T = a.n_groups, Tq = a.t_q;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fi = lane & 15, kk = lane >> 4;
    const float* keys = a.keys + ((int64_t)(a.layer0 + li) * a.capacity_groups) * HD;
    const double* qtok = a.ws_qtok + (int64_t)li * Tq * HD;

    __shared__ double wsum[kBlock / 64];
    const QueryNorm2<kBlock> norm(a, li, HD);

    double colsum = 0.0, nk2 = 0.0;
    if constexpr (MOST <= 2) {
        gemm_rows<MOST, NG>(a, As, Bs, qtok, keys, 0, n0, li, colsum, nk2);
    } else {
        for (int m0 = 0; m0 < Tq; m0 += kGemmM) {
            const int mt = (min(kGemmM, Tq - m0) + 15) >> 4;
            switch (mt) {  // uniform; halves of tiles need an even number of them
                case 1:
                    if constexpr (NG == 4) {
                        gemm_rows<1, NG>(a, As, Bs, qtok, keys, m0, n0, li, colsum, nk2);
                        break;
                    }
                    [[fallthrough]];
                case 2: gemm_rows<2, NG>(a, As, Bs, qtok, keys, m0, n0, li, colsum, nk2); break;
                case 3:
                    if constexpr (NG == 4) {
                        gemm_rows<3, NG>(a, As, Bs, qtok, keys, m0, n0, li, colsum, nk2);
                        break;
                    }
                    [[fallthrough]];
                default: gemm_rows<4, NG>(a, As, Bs, qtok, keys, m0, n0, li, colsum, nk2); break;
            }
        }
    }
    norm.put(wsum);
    // lanes fi, 16 + fi, 32 + fi, 48 + fi hold the partial sums of group n0 + 16 * tile + fi
    colsum = rows16_sum_f64(colsum);
    nk2 = rows16_sum_f64(nk2);
    __shared__ double other[NG == 2 ? 32 : 1];  // of the waves with the upper half of the tokens
    if (NG == 2 && wave >= 2 && kk == 0) other[(wave - 2) * 16 + fi] = colsum;
    __syncthreads();
    const int t = n0 + wave * 16 + fi;
    if (wave < NG && kk == 0 && t < T) {
        if (NG == 2) colsum += other[wave * 16 + fi];
        double s = colsum / (double)Tq;
        if (a.sim == TOM_SIM_COSINE) {
            s = s / (fmax(sqrt(total_of<kBlock / 64>(wsum)), 1e-12) * fmax(sqrt(nk2), 1e-12));
        }
        a.scores[(int64_t)li * a.score_stride + t] = (float)s;
    }
}

// The same contraction for launches of few units of 16 groups, or of few tokens on long keys (split_tiles in oqm_dispatch.h), where the 64 x 64 form
// leaves compute units idle and each of its few workgroups walks the whole contraction through
// barriers (1.2 us per 32 channels).  Unit of work = (layer, 16
// consecutive groups), all query tokens in passes of 16 * MT: the eight waves of a workgroup split the contraction,
// wave w taking the blocks w, w + 8, ... of 16 channels, and add their tiles up in LDS at the end.
// Operands go from memory straight into the MFMA registers: the order of a contraction is free,
// so lane (fi, kk) takes channels 4 kk .. 4 kk + 3 of a block for its four MFMA steps and every load is 16 bytes
// wide; kAhead blocks are requested before the first is used (four: no faster, one at a time: 3 to 8 us slower).
constexpr int kSplitWaves = 8, kSplitThreads = 64 * kSplitWaves, kAhead = 2;

template <int MT>
__global__ void __launch_bounds__(kSplitThreads) score_token_split_kernel(const ScoreArgs a) {
    __shared__ double red[kSplitWaves][2 * 256];  // two 16 x 16 tiles of every wave
    __shared__ double col[2][kSplitWaves][16];
    __shared__ double wsum[kSplitWaves];
    request(a);
    const int unit = (int)(blockIdx.x & 7u) * a.gemm_units_per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= a.gemm_units) return;  // uniform per workgroup
    const int li = div_by(unit, a.gemm_tiles_per_layer, a.inv_gemm_tiles_per_layer);
    const int n0 = (unit - li * a.gemm_tiles_per_layer) * 16;
    const int HD = a.n_kv_heads * a.head_dim;
    const int T = a.n_groups, Tq = a.t_q;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = lane & 15, kk = lane >> 4;
    const int blocks = (HD + 15) >> 4;
    // groups past T and tokens past T_q repeat the last one and are dropped at the end
    const float* const key = a.keys + ((int64_t)(a.layer0 + li) * a.capacity_groups + min(n0 + fi, T - 1)) * HD;
    const double* const qtok = a.ws_qtok + (int64_t)li * Tq * HD;
    const QueryNorm2<kSplitThreads> norm(a, li, HD);

    double csum = 0.0, nk2 = 0.0;
    for (int m0 = 0; m0 < Tq; m0 += 16 * MT) {
        const double* row[MT];
        f64x4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            row[m] = qtok + (int64_t)min(m0 + m * 16 + fi, Tq - 1) * HD;
            acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
        }
        for (int b0 = wave; b0 < blocks; b0 += kAhead * kSplitWaves) {
            f64x2 ra[kAhead][MT][2];
            f32x4 rb[kAhead];
#pragma unroll
            for (int p = 0; p < kAhead; ++p) {
                const int b = b0 + p * kSplitWaves;
                if (b < blocks) {  // uniform
                    const int k = min(b * 16 + kk * 4, HD - 4);  // HD is a multiple of 8
                    rb[p] = *reinterpret_cast<const f32x4*>(key + k);
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        ra[p][m][0] = *reinterpret_cast<const f64x2*>(row[m] + k);
                        ra[p][m][1] = *reinterpret_cast<const f64x2*>(row[m] + k + 2);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < kAhead; ++p) {
                const int b = b0 + p * kSplitWaves;
                if (b >= blocks) break;  // uniform
                if (b * 16 + kk * 4 >= HD) {  // half a block: the upper lanes re-read the last channels
                    rb[p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int m = 0; m < MT; ++m) ra[p][m][0] = ra[p][m][1] = f64x2{0.0, 0.0};
                }
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const double bv = (double)rb[p][st];
                    if (m0 == 0) nk2 = fma(bv, bv, nk2);
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[p][m][st >> 1][st & 1], bv, acc[m], 0, 0, 0);
                }
            }
        }
        if (m0 == 0) norm.put(wsum);  // read behind the barriers below
        // add up the waves, two tiles at a time: thread (u, e) owns element e = v * 64 + lane of tile m + u
#pragma unroll
        for (int m = 0; m < MT; m += 2) {
            if (m0 + m > 0) __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (m + u < MT) red[wave][u * 256 + v * 64 + lane] = acc[m + u < MT ? m + u : 0][v];
            __syncthreads();
            const int j = m0 + (m + (tid >> 8)) * 16 + mfma_d_row(lane, (tid >> 6) & 3);
            if (m + (tid >> 8) < MT && j < Tq) {
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < kSplitWaves; ++w) sum += red[w][tid];
                csum += sum;
                if (a.token_scores && n0 + fi < T) a.token_scores[((int64_t)li * Tq + j) * T + n0 + fi] = (float)sum;
            }
        }
    }
    const double nq = sqrt(total_of<kSplitWaves>(wsum));
    // lanes fi, 16 + fi, 32 + fi, 48 + fi hold parts of group n0 + fi
    csum = rows16_sum_f64(csum);
    nk2 = rows16_sum_f64(nk2);
    if (kk == 0) {
        col[0][wave][fi] = csum;
        col[1][wave][fi] = nk2;
    }
    __syncthreads();
    if (tid < 16 && n0 + tid < T) {
        double s = 0.0, n2 = 0.0;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) {
            s += col[0][w][tid];
            n2 += col[1][w][tid];
        }
        s = s / (double)Tq;
        if (a.sim == TOM_SIM_COSINE) s = s / (fmax(nq, 1e-12) * fmax(sqrt(n2), 1e-12));
        a.scores[(int64_t)li * a.score_stride + n0 + tid] = (float)s;
    }
}

// Fold and split contraction in one launch, for small launches (fold_tiles in oqm_dispatch.h): the query is folded where it enters the MFMA
// registers.  Lane (fi, kk) takes token fi of a tile and channels 8 kk .. 8 kk + 7 of a block of 32, loads 16 bytes of each of the r query heads that
// its KV head stands for, and averages them on the vector pipe; blocks go round the eight waves, pieces past the end of the query are read as zero.
// Every workgroup of a layer reads its question, at 2 r bytes an element against the 8 of a folded one, so the launch of the fold (4.5 us and more)
// is saved for nothing up to four heads of 16 bits; with more the conversions and the loads of a block in RH heads at a time cost more than they save.  Bound by
// latency: load, convert, MFMA, two blocks a wave at 512 channels.  Whole question on the device at 4 groups, bf16, before / now: one layer x 64
// groups x 1 head of 64 x 13 tokens 11.6 / 8.7 us, 28 x 280 x 1 of 128 x 64 18.9 / 13.5, 16 x 512 x 12 heads on 3 of 96 x 30 19.1 / 14.8, 28 x 130 x
// 16 on 4 of 128 x 64 24.7 / 19.5, 28 x 100 x 10 on 5 of 256 x 64 43.8 / 29.6, 28 on 4 of 128, one layer x 256 x 16 13.0 / 11.9. MT tiles of 16
// tokens a pass: 78 to 128 registers with one or two, 144 to 223 with three or four (one workgroup a compute unit).
struct TokenFold {
    uint32_t inv_head_dim;
};

__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, uint32_t off, Raw8<In_bf16>& x) {
    x.a = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, uint32_t off, Raw8<In_f16>& x) {
    x.a = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, uint32_t off, Raw8<In_f32>& x) {
    x.a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    x.b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 16, 0));
}

// Dynamic LDS with the cosine: H_k*d doubles, the sums of the folded query over its tokens.
template <typename QT, int MT, int RH>
__global__ void __launch_bounds__(kSplitThreads) score_token_fold_kernel(const ScoreArgs a, const TokenFold f) {
    constexpr int EB = elem_bytes<QT>::value;
    constexpr uint32_t kOutside = 0x80000000u;  // an offset past the end of any query (fold_tiles)
    __shared__ double red[kSplitWaves][2 * 256];  // two 16 x 16 tiles of every wave
    __shared__ double col[2][kSplitWaves][16];
    __shared__ double wsum[kSplitWaves];
    extern __shared__ __align__(16) double qsum[];
    request(a);
    const int unit = (int)(blockIdx.x & 7u) * a.gemm_units_per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= a.gemm_units) return;  // uniform per workgroup
    const int li = div_by(unit, a.gemm_tiles_per_layer, a.inv_gemm_tiles_per_layer);
    const int n0 = (unit - li * a.gemm_tiles_per_layer) * 16;
    const int d = a.head_dim, HD = a.n_kv_heads * d;
    const int T = a.n_groups, Tq = a.t_q, r = a.n_q_heads / a.n_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = lane & 15, kk = lane >> 4;
    const int blocks = (HD + 31) >> 5;
    const bool norm = a.sim == TOM_SIM_COSINE;
    // groups past T repeat the last one and are dropped at the end
    const float* const key = a.keys + ((int64_t)(a.layer0 + li) * a.capacity_groups + min(n0 + fi, T - 1)) * HD;
    const uint32_t row_bytes = (uint32_t)d * EB, head_bytes = (uint32_t)Tq * row_bytes, layer_bytes = (uint32_t)a.n_q_heads * head_bytes;
    const __amdgpu_buffer_rsrc_t q = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(a.q)) + (uint64_t)li * layer_bytes, 0, (int)layer_bytes, 0x00020000);
    const double inv_r = 1.0 / (double)r;

    double csum = 0.0, nk2 = 0.0;
    for (int m0 = 0; m0 < Tq; m0 += 16 * MT) {
        f64x4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
        for (int b = wave; b < blocks; b += kSplitWaves) {
            const int k = b * 32 + kk * 8;
            const bool in = k < HD;
            const int h = div_by((uint32_t)k, (uint32_t)d, f.inv_head_dim);
            const uint32_t first = in ? (uint32_t)(h * r) * head_bytes + (uint32_t)(k - h * d) * EB : kOutside;
            double qt[MT][8];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int i = 0; i < 8; ++i) qt[m][i] = 0.0;
            f32x4 rb[2];
            for (int g0 = 0; g0 < r; g0 += RH) {
                Raw8<QT> raw[MT][RH];
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int g = 0; g < RH; ++g) {
                        const int j = m0 + m * 16 + fi;
                        load_row(q, j < Tq && g0 + g < r ? first + (uint32_t)(g0 + g) * head_bytes + (uint32_t)j * row_bytes : kOutside, raw[m][g]);
                    }
                if (g0 == 0) {
                    const float* p = key + min(k, HD - 8);
                    rb[0] = *reinterpret_cast<const f32x4*>(p);
                    rb[1] = *reinterpret_cast<const f32x4*>(p + 4);
                }
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int g = 0; g < RH; ++g) {
                        float x[8];
                        widen(raw[m][g], x);
#pragma unroll
                        for (int i = 0; i < 8; ++i) qt[m][i] += (double)x[i];
                    }
            }
            if (!in) rb[0] = rb[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double bv = (double)rb[i >> 2][i & 3];
                if (m0 == 0) nk2 = fma(bv, bv, nk2);
                double s = 0.0;
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    qt[m][i] *= inv_r;
                    s += qt[m][i];
                    acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(qt[m][i], bv, acc[m], 0, 0, 0);
                }
                if (norm) {  // uniform; a block's channels are this wave's alone
                    s = row16_sum_f64(s);
                    if (fi == 0 && in) qsum[k + i] = m0 == 0 ? s : qsum[k + i] + s;
                }
            }
        }
        // add up the waves, two tiles at a time: thread (u, e) owns element e = v * 64 + lane of tile m + u
#pragma unroll
        for (int m = 0; m < MT; m += 2) {
            if (m0 + m > 0) __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (m + u < MT) red[wave][u * 256 + v * 64 + lane] = acc[m + u < MT ? m + u : 0][v];
            __syncthreads();
            const int j = m0 + (m + (tid >> 8)) * 16 + mfma_d_row(lane, (tid >> 6) & 3);
            if (m + (tid >> 8) < MT && j < Tq) {
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < kSplitWaves; ++w) sum += red[w][tid];
                csum += sum;
                if (a.token_scores && n0 + fi < T) a.token_scores[((int64_t)li * Tq + j) * T + n0 + fi] = (float)sum;
            }
        }
    }
    if (norm) {  // the sums of all waves were put in front of the last barrier
        double sq = 0.0;
        const double share = 1.0 / (double)Tq;
        for (int e = tid; e < HD; e += kSplitThreads) {
            const double qb = qsum[e] * share;
            sq = fma(qb, qb, sq);
        }
        put_wave_sum(sq, wsum);
    }
    // lanes fi, 16 + fi, 32 + fi, 48 + fi hold parts of group n0 + fi
    csum = rows16_sum_f64(csum);
    nk2 = rows16_sum_f64(nk2);
    if (kk == 0) {
        col[0][wave][fi] = csum;
        col[1][wave][fi] = nk2;
    }
    __syncthreads();
    if (tid < 16 && n0 + tid < T) {
        double s = 0.0, n2 = 0.0;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) {
            s += col[0][w][tid];
            n2 += col[1][w][tid];
        }
        s = s / (double)Tq;
        if (norm) s = s / (fmax(sqrt(total_of<kSplitWaves>(wsum)), 1e-12) * fmax(sqrt(n2), 1e-12));
        a.scores[(int64_t)li * a.score_stride + n0 + tid] = (float)s;
    }
}

}  // namespace

static hipError_t launch_query_fold(const ScoreArgs& a, bool want_tokens, hipStream_t s) {
    if (a.n_layers == 0) return hipSuccess;
    const int parts = fold_parts(a, want_tokens);
    const dim3 grid(a.n_kv_heads * parts, a.n_layers), block(kFoldThreads);
    auto go = [&](auto qt) {
        typedef decltype(qt) QT;
        if (want_tokens) launch(query_fold_kernel<QT, true>, grid, block, 0, s, a, parts);
        else launch(query_fold_kernel<QT, false>, grid, block, 0, s, a, parts);
        return hipGetLastError();
    };
    switch (a.q_dtype) {
        case TOM_F32: return go(In_f32{});
        case TOM_BF16: return go(In_bf16{});
        case TOM_F16: return go(In_f16{});
        default: return hipErrorInvalidValue;
    }
}

// Calls go with the pieces of 4 * W key channels that a lane loads together and what they leave, as types, and the bytes of a staged q-bar: one trip
// of up to eight pieces, or the fewest equal trips if they leave nothing.  Exactly as many pieces as the key has instead of two, four or eight: 28
// layers x 1024 groups x 5 heads of 128 24.2 -> 21.1 us (whole question, k = 1), 3 of 96 18.5 -> 17.3.
template <int W, typename GO>
static hipError_t with_pieces(int HD, GO go) {
    const int pieces = (HD + 4 * W - 1) / (4 * W), trips = (pieces + kScoreChunks - 1) / kScoreChunks;
    const bool whole = HD % (4 * W * trips) == 0;
    auto with = [&](auto ch, auto rest) {
        constexpr int trip = 4 * W * decltype(ch)::value;
        go(ch, rest, (size_t)((HD + trip - 1) / trip * trip) * sizeof(double));
        return hipGetLastError();
    };
    // 32 lanes take keys of at least eight pieces: eight whole ones, or several trips of five to eight
    constexpr bool long_keys = W == 32;
    auto each = [&](auto ch) {
        if (whole) return with(ch, std::integral_constant<Rest, kNoRest>{});
        if constexpr (!long_keys) {
            if (trips == 1) return with(ch, std::integral_constant<Rest, kLastPiece>{});
        }
        return with(std::integral_constant<int, kScoreChunks>{}, std::integral_constant<Rest, kAnyPiece>{});
    };
    const int per_trip = (pieces + trips - 1) / trips;
    if constexpr (!long_keys) {
        switch (per_trip) {
            case 1: return each(std::integral_constant<int, 1>{});
            case 2: return each(std::integral_constant<int, 2>{});
            case 3: return each(std::integral_constant<int, 3>{});
            case 4: return each(std::integral_constant<int, 4>{});
        }
    }
    switch (per_trip) {
        case 5: return each(std::integral_constant<int, 5>{});
        case 6: return each(std::integral_constant<int, 6>{});
        case 7: return each(std::integral_constant<int, 7>{});
        default: return each(std::integral_constant<int, 8>{});
    }
}

hipError_t launch_score_mean_query(const ScoreArgs& a, hipStream_t s) {
    if (a.n_layers == 0 || a.n_groups == 0) return hipSuccess;
    const int HD = a.n_kv_heads * a.head_dim;
    FoldSplit f{};
    f.slots = fold_slots(a);
    if (f.slots > 0) {
        f.inv_slots = reciprocal_u32(f.slots);
        f.inv_lanes_per_row = reciprocal_u32((uint32_t)a.head_dim / 8u);
        f.inv_head_dim = reciprocal_u32((uint32_t)a.head_dim);
        const int lpr = a.head_dim / 8;
        f.waves = rows_divide_a_wave(lpr) && f.slots * lpr % 64 == 0 ? f.slots * lpr / 64 : 0;
        const dim3 grid((a.n_groups + kFoldThreads / 16 - 1) / (kFoldThreads / 16), a.n_layers), block(kFoldThreads);
        return with_pieces<16>(HD, [&](auto ch, auto rest, size_t lds) {
            constexpr int CH = decltype(ch)::value;
            constexpr Rest REST = decltype(rest)::value;
            if (a.q_dtype == TOM_F32) launch(score_fold_query_kernel<In_f32, CH, REST>, grid, block, lds, s, a, f);
            else if (a.q_dtype == TOM_BF16) launch(score_fold_query_kernel<In_bf16, CH, REST>, grid, block, lds, s, a, f);
            else launch(score_fold_query_kernel<In_f16, CH, REST>, grid, block, lds, s, a, f);
        });
    }
    if (hipError_t e = launch_query_fold(a, false, s)) return e;
    auto go = [&](auto lanes) {
        constexpr int W = decltype(lanes)::value, per_block = kBlock / W;
        const dim3 grid((a.n_groups + per_block - 1) / per_block, a.n_layers);
        return with_pieces<W>(HD, [&](auto ch, auto rest, size_t lds) {
            constexpr int CH = decltype(ch)::value;
            constexpr Rest REST = decltype(rest)::value;
            if (keys_past_caches(a)) launch(score_mean_query_kernel<W, CH, REST, true>, grid, dim3(kBlock), lds, s, a);
            else launch(score_mean_query_kernel<W, CH, REST, false>, grid, dim3(kBlock), lds, s, a);
        });
    };
    // long keys in one trip of 512-byte pieces: 28 x 1024 groups x 8 heads of 128 39.6 -> 35.9 us, 700 x 8 of 256 47.5 -> 45.1, but
    // 1024 x 5 of 128 (two trips of five 256-byte pieces) 23.1 -> 25.4
    return HD >= 1024 ? go(std::integral_constant<int, 32>{}) : go(std::integral_constant<int, 16>{});
}

hipError_t launch_score_token_gemm(const ScoreArgs& args, hipStream_t s) {
    if (args.n_layers == 0 || args.n_groups == 0) return hipSuccess;
    ScoreArgs a = args;
    const int folded = fold_tiles(a);
    if (!folded)
        if (hipError_t e = launch_query_fold(args, true, s)) return e;
    const int tiles = folded ? folded : split_tiles(a);
    const int width = tiles > 0 ? 16 : gemm_width(a);
    a.gemm_tiles_per_layer = (a.n_groups + width - 1) / width;
    a.inv_gemm_tiles_per_layer = reciprocal_u32((uint32_t)a.gemm_tiles_per_layer);
    const int64_t units = (int64_t)a.gemm_tiles_per_layer * a.n_layers;
    if (units > 0x7fffffffLL - 8) return hipErrorInvalidValue;  // 2^25 tiles x 65535 layers at most: never
    a.gemm_units = (int32_t)units;
    a.gemm_units_per_xcd = (int32_t)((units + 7) / 8);
    const dim3 grid(8u * (unsigned)a.gemm_units_per_xcd);
    if (folded) {
        const TokenFold f{reciprocal_u32((uint32_t)a.head_dim)};
        const size_t lds = a.sim == TOM_SIM_COSINE ? (size_t)a.n_kv_heads * a.head_dim * sizeof(double) : 0;
        const int r = a.n_q_heads / a.n_kv_heads;
        auto go = [&](auto qt, auto mt, auto rh) {
            launch(score_token_fold_kernel<decltype(qt), decltype(mt)::value, decltype(rh)::value>, grid, dim3(kSplitThreads), lds, s, a, f);
            return hipGetLastError();
        };
        auto heads = [&](auto qt, auto mt) {
            if (r == 1) return go(qt, mt, std::integral_constant<int, 1>{});
            if constexpr (elem_bytes<decltype(qt)>::value == 2) {
                if (r > 2) return go(qt, mt, std::integral_constant<int, 4>{});
            }
            return go(qt, mt, std::integral_constant<int, 2>{});
        };
        auto type = [&](auto mt) {
            if (a.q_dtype == TOM_F32) return heads(In_f32{}, mt);
            return a.q_dtype == TOM_BF16 ? heads(In_bf16{}, mt) : heads(In_f16{}, mt);
        };
        switch (folded) {
            case 1: return type(std::integral_constant<int, 1>{});
            case 2: return type(std::integral_constant<int, 2>{});
            case 3: return type(std::integral_constant<int, 3>{});
            default: return type(std::integral_constant<int, 4>{});
        }
    }
    switch (tiles) {
        case 0:
            if (width == kGemmN / 2) {
                if (a.t_q <= 32) launch(score_token_gemm_kernel<2, 2>, grid, dim3(kBlock), 0, s, a);
                else launch(score_token_gemm_kernel<4, 2>, grid, dim3(kBlock), 0, s, a);
                break;
            }
            if (a.t_q <= 16) launch(score_token_gemm_kernel<1, 4>, grid, dim3(kBlock), 0, s, a);
            else if (a.t_q <= 32) launch(score_token_gemm_kernel<2, 4>, grid, dim3(kBlock), 0, s, a);
            else launch(score_token_gemm_kernel<4, 4>, grid, dim3(kBlock), 0, s, a);
            break;
        case 1: launch(score_token_split_kernel<1>, grid, dim3(kSplitThreads), 0, s, a); break;
        case 2: launch(score_token_split_kernel<2>, grid, dim3(kSplitThreads), 0, s, a); break;
        case 3: launch(score_token_split_kernel<3>, grid, dim3(kSplitThreads), 0, s, a); break;
        default: launch(score_token_split_kernel<4>, grid, dim3(kSplitThreads), 0, s, a);
    }
    return hipGetLastError();
}
}  // namespace oqm
