// The rules by which the host side chooses between forms of a kernel that give the same results:
// plain functions of sizes and addresses, so that the CPU tests can ask them directly.
#pragma once

#include "oqm_common.h"

namespace oqm {

// Two byte ranges share no memory.
inline bool apart(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x + a_bytes <= y || y + b_bytes <= x;
}

// Bytes from the first to the last score of `n_layers` rows.
inline uint64_t score_span(int64_t stride, int n_layers, int n_groups) {
    return sizeof(float) * ((uint64_t)(n_layers - 1) * (uint64_t)stride + (uint64_t)n_groups);
}

// ---- mean-query score: keys past the caches --------------------------------------------------
// From 100 MB up the keys of a call are a good part of the last-level cache (256 MB), and read through it they push out the codes of the next gather.
// Past the caches they are read again from memory for the next question about the same store, which costs less than it looks, since 100 MB of keys do
// not survive a question whole either.  28 layers x 512 channels, us, through / past, one store asked in a row and three in turn.  Scores alone: 100
// MB 20.8 / 20.2, 23.2 / 21.9; 126 24.7 / 24.0, 27.1 / 25.6; 172 30.5 / 30.3, 34.5 / 32.1; 206 34.9 / 35.2, 40.1 / 37.0; 300 51.1 / 48.5, 55.0 /
// 50.7.  Whole question at 4 selected groups: 100 33.6 / 34.2, 40.7 / 34.8; 126 38.9 / 39.4, 46.1 / 39.9; 172 44.6 / 46.0, 53.7 / 46.5; 206 50.6 /
// 50.6, 58.8 / 51.1; at 1 172 39.0 / 39.6, 44.7 / 41.1; at 16 126 61.8 / 60.7, 75.1 / 64.9; 172 79.6 / 67.1, 82.4 / 72.3; at 64 172 198 / 192, 203 /
// 195.  The most lost: 8 heads of 128, 172 MB, 4 groups 44.4 / 46.5 (in turn 51.7 / 46.3).  Smaller ones in turn: 57 MB 14.9 / 15.8 (scores alone),
// 86 19.9 / 20.5.
constexpr int64_t kKeysPastCaches = 100000000;
inline bool keys_past_caches(const ScoreArgs& a) {
    return (int64_t)a.n_layers * a.n_groups * a.n_kv_heads * a.head_dim * (int64_t)sizeof(float) >= kKeysPastCaches;
}

// ---- mean-query score: the query is folded inside the score kernel -----------------------
constexpr int kFoldThreads = 512;

// Row slots per KV head of score_fold_query_kernel, or 0: the fold is a launch of its own. Folding inside the score kernel saves a launch (about 4 us
// on the device) and costs every workgroup the serial sum over the rows of a slot, 0.15 us a row, more once workgroups share compute units: line at
// rows x (workgroups + 168).  Whole question at k = 1, fused / separate: 28 heads on 4 of 128, 2 workgroups x 24 tokens (21 rows) 10.5 / 11.5 us, 32
// (28) 11.6 / 11.6, 48 13.9 / 11.3; 64 workgroups x 16 tokens 10.7 / 11.6, 24 12.0 / 10.9; 56 heads on 8 of 80, 6 workgroups x 16 tokens (19 rows)
// 12.1 / 12.7, 24 (28) 13.2 / 12.4; 12 on 3 of 96, 325 workgroups x 24 tokens (7 rows) 14.4 / 14.7, 32 (10) 16.4 / 14.6; 224 workgroups x 32 tokens
// (10 rows) 10.0 / 11.6, 28 on 4 of 128 224 x 11 tokens (10 rows) 11.3 / 11.3, 12 (11) 12.1 / 11.3.  In several rounds of the chip it is the bytes of
// the query that count: 28 heads on 4 of 128, 896 workgroups x 1 token 20.0 / 20.1, x 4 21.1 / 20.2, 1764 x 1 32.0 / 32.3, x 2 32.6 / 32.2; 6 on 3 of
// 128, 2912 x 1 40.8 / 40.9, x 4 44.4 / 41.0. A compute unit holds two workgroups of up to 128 registers: 16-bit queries at any key (77 to 110),
// float32 ones at keys of up to five pieces of 64 channels (110 to 128; six to eight 130 to 140).  A launch of more runs the serial fold again in a
// second round.  Every workgroup of a layer reads its question, so an XCD reads that of every layer with eight workgroups or more, besides an eighth
// of the keys: a float32 question that the L2 (4 MiB) cannot hold so keeps the limits of one workgroup a compute unit, and rows x (workgroups + 160).
// 28 layers, MB of question and keys an XCD, us fused / separate: 4 heads of 64, 280 workgroups 3.9 6.8 / 7.0, 4.4 7.7 / 7.0, 4.8 10.1 / 7.0; 448 4.1
// 6.9 / 7.4, 4.6 8.0 / 7.4; 5 of 64 448 4.4 7.9 / 8.0, 4.9 9.3 / 8.1; 3 of 96 448 4.2 7.5 / 8.3, 4.8 9.2 / 8.3; 224 x 10 rows 4 of 64 5.5 10.0 / 6.7,
// 14 layers x 16 (3.2) 5.9 / 6.7, 4 of 128 (4.1) 8.2 / 7.6.  Fold and scores in a graph, fused / separate: float32, 270 / 448 / 512 workgroups x 1
// token, one head of 64 4.7 / 6.4 us, 4.8 / 6.8, 4.8 / 6.7; 5 heads of 64 6.0 / 7.3, 6.2 / 8.0, 6.2 / 8.0, x 16 tokens 6.7 / 7.3, 6.9 / 7.9, 6.9 /
// 8.0; 3 of 128 (six pieces) x 4 7.8 / 7.5, 7.9 / 8.2, 8.0 / 8.3; 4 of 128 x 1 8.4 / 7.9, 8.5 / 8.7, 8.6 / 9.0, x 16 9.6 / 7.9, 12.1 / 8.9, 11.8 /
// 9.8, 256 x 1 6.9 / 9.2; one head of 64, 896 x 64 17.9 / 9.6. 16-bit: one head of 64, 512 workgroups 6.7 / 8.4, 544 9.6 / 8.7, 896 x 64 tokens 13.2
// / 9.7; where the keys are longer they hide it: 4 heads of 128, 768 x 1 14.5 / 16.0. Scores that share memory with the query need the separate fold
// at any size: in one launch some workgroups write scores while others still read the query.
inline uint32_t fold_slots(const ScoreArgs& a) {
    constexpr int64_t kFusedRows = 3930, kFusedRowsPastL2 = 3800, kFusedWork = 6500000, kL2 = 4 << 20, kXcds = 8;
    const uint32_t slots = (uint32_t)(kFoldThreads / (a.head_dim / 8) / a.n_kv_heads);
    if (slots == 0) return 0;
    const int64_t layer_blocks = (a.n_groups + kFoldThreads / 16 - 1) / (kFoldThreads / 16), blocks = layer_blocks * a.n_layers;
    const int64_t rows = (int64_t)(a.n_q_heads / a.n_kv_heads) * a.t_q;
    const int64_t query = rows * a.n_kv_heads * a.head_dim;  // elements of a layer
    const int channels = a.n_kv_heads * a.head_dim;
    const bool is_f32 = a.q_dtype == TOM_F32;
    bool one = false;  // float32: one workgroup a compute unit
    if (is_f32) {
        const int64_t readers = layer_blocks < kXcds ? layer_blocks : kXcds;
        one = channels > 5 * 64 || query * readers + (int64_t)a.n_groups * channels > kL2 / 4 * kXcds / a.n_layers;
    }
    if ((rows + slots - 1) / slots > (one ? kFusedRowsPastL2 / (blocks + 160) : kFusedRows / (blocks + 168))) return 0;
    if (blocks > 512 && query > kFusedWork / (blocks + 64)) return 0;
    if (is_f32 ? blocks > (one ? 256 : 512) : blocks > 512 && channels < 256) return 0;
    const uint64_t query_bytes = (uint64_t)query * (uint64_t)a.n_layers * (is_f32 ? 4u : 2u);
    return apart(a.q, query_bytes, a.scores, score_span(a.score_stride, a.n_layers, a.n_groups)) ? slots : 0u;
}

// ---- query fold of its own -------------------------------------------------------------------
// Workgroups per KV head of query_fold_kernel: one per 64 channels where those divide the head and the launch stays within one round of the chip (two
// workgroups a compute unit), or where a row slot of a whole head would fold more than three tokens one after the other; otherwise one.  Fold and
// scores of 28 layers x 64 groups in a graph, parts / one: 5 heads of 256 (560 workgroups), per-token scores of 1 query token 13.9 / 12.0 us, 33 30.1
// / 28.2, mean query of 33 11.0 / 8.5; 8 of 256 (896) 1 17.6 / 15.2, 33 39.1 / 37.0, 64 54.6 / 56.3, mean of 64 14.8 / 10.3; 4 of 512 (896) 10 21.0 /
// 19.7, 64 54.8 / 57.8, mean of 64 14.8 / 12.1; 4 of 256 (448) 10 13.2 / 13.5, 64 34.1 / 35.2, mean of 64 10.0 / 12.1.
inline int fold_parts(const ScoreArgs& a, bool want_tokens) {
    const int64_t parts = a.head_dim / 64;
    if (a.head_dim % 64 != 0) return 1;
    return parts * a.n_kv_heads * a.n_layers <= 512 || (want_tokens && a.t_q > 3 * (kFoldThreads / (a.head_dim / 8))) ? (int)parts : 1;
}

// ---- per-token scores: the contraction is split over the waves of a workgroup -------------
constexpr int kGemmN = 64;  // groups of a unit of the 64 x 64 form
// More than 512 units of 16 groups (`wide`: of 64): whether up to 16 query tokens split the contraction.  The 64 x 64 form is bound by its chain of
// chunks, a barrier and a load latency for 32 channels, with one or two workgroups a compute unit; its time steps up behind 256 units of 64 (1024 of
// 16). The split form steps up with every 256 units, a workgroup more on each compute unit, and grows with the tokens, which it reads once a unit.
// So per step up to c - k / channels tokens.  Fold and scores, 64 x 64 form / this, at the last tokens kept and some behind them:
//   513 to 768 units: 256 channels x 8 tokens 0.98 to 0.99, x 15 11.1 / 11.7; 288 x 10 12.1 / 11.6; 320 x 13 0.95; 400 x 15 15.0 / 13.6; 512 x 16
//     0.97; 1024 x 16 0.95
//   769 to 1024 (with more than 256 units of 64 as the next row: 1012 of 256 x 1 13.1 / 11.1): 256 x 1 1.00 to 1.03; 288 x 3 12.1 / 11.6; 320 x 5
//     0.97, x 8 12.8 / 13.4; 480 x 6 15.9 / 15.1; 512 x 7 0.98, x 12 16.3 / 17.9; 1024 x 9 0.97, x 14 25.1 / 27.1; 1280 x 11 1.00, x 14 1.07; 2048 x 12
//     0.83 (again 1.02), x 14 0.87 (1.07).  Keys of 1280 channels and more go on by a second line.
//   1025 to 1280: 256 x 7 0.98, x 12 1.04; 320 x 9 15.2 / 14.3; 400 x 10 0.95; 512 x 11 0.97, x 14 1.01; 1024 x 11 0.92, x 15 1.01; 1280 x 13 1.02 to 1.06
//     (0.93), x 16 1.12 to 1.16 (1.03); 2048 x 14 0.92 (0.96)
//   1281 to 1536: 256 x 1 13.3 / 14.0; 320 x 1 1.00, x 5 1.04; 400 x 4 18.1 / 16.6; 512 x 5 19.7 / 18.7, x 8 1.03; 640 x 6 24.0 / 22.7; 768 x 8 1.00;
//     1024 x 9 0.96, x 11 1.02; 1280 x 9 1.04 to 1.07 (0.95), x 11 1.13 (1.03); 2048 x 10 0.94 (0.98), x 14 1.03 (1.11)
//   1537 to 1792: 512 x 1 1.01; 768 x 3 1.00, x 7 1.06; 1024 x 3 38.6 / 34.5, x 5 38.5 / 35.6; 1280 x 5 1.00 to 1.02 (0.96), x 9 1.16 (1.08); 2048 x 7
//     0.96 (1.02), x 11 1.05 (1.16)
//   1793 to 2048: 512 x 2 1.12; 1024 x 1 40.3 / 37.6, x 2 1.02; 1280 x 1 0.87 to 0.94 (0.79 to 0.98), x 5 1.01 to 1.07; 2048 x 3 0.93 (0.78 to 0.99), x
//     7 1.00 to 1.03 (0.89 to 1.14)
// Three stores in turn (the same question again, where it differs by more than 4 %; 1024 channels from 1537 units on gain 4 to 8 % less again).
inline bool one_tile_splits(int64_t units, int64_t wide, int t_q, int channels) {
    static constexpr struct { int c, k, channels; } kLine[] = {{40, 8192, 256}, {11, 1800, 288}, {15, 1900, 256}, {12, 3000, 352}, {9, 4000, 576}, {6, 5000, 256}};  // three to eight units a compute unit
    int64_t step = (units + 255) / 256 - 3;
    if (step == 1 && wide > 256) step = 2;
    if (t_q > 16 || step < 0 || step > 5 || channels < kLine[step].channels) return false;
    if (step == 1 && (int64_t)(16 - t_q) * channels >= 6400) return true;
    return (int64_t)(kLine[step].c - t_q) * channels >= kLine[step].k;
}

// Tiles of 16 query tokens per pass of score_token_split_kernel (1 to 4), or 0: the 64 x 64 form.
//   up to 512 units of 16 groups, two a compute unit: a whole question on the device (fold, this, top-k, gather of 4 groups) at 4 heads of 128, this
//     / 64 x 64 form: 1 layer x 256 groups x 32 tokens 18.1 / 28.0 us, x 64 25.8 / 39.3; 8 x 1024 (512 units) x 32 25.3 / 31.0; but 28 x 400 (700
//     units) x 32 33.0 / 33.0, x 64 55.2 / 45.9: from three units a compute unit on the query block is read too often
//   equal passes of up to four tiles to 256 units, up to three above: four take 144 registers, one workgroup a compute unit, three 118, two
//     workgroups.  Fold and scores at 448 to 512 units, equal passes of three / passes of four / 64 x 64 form: one head of 64 x 65 tokens 14.5 / 18.0
//     / 15.8 us, x 1024 92 / 117 / 107; 4 heads of 128 x 65 36 / 45 / 46, x 1024 370 / 390 / 470
//   one tile on keys of 256 channels and more goes on beyond (one_tile_splits)
//   two and three tiles whose last is mostly empty (up to 5 t <= 64 tiles; its lanes re-read one row here, the 64 x 64 form multiplies them) go on as
//     well on keys of 512 channels and more, where the 64 x 64 form would leave a third of one round of the chip idle, up to 168 units of 64, or,
//     three tiles, two fifths of two, 257 to 308.  Fold and scores, 64 x 64 form / this, at 17 / 25 / 33 / 38 tokens: 28 layers x 384 groups of 512
//     channels (168) 21.3 / 18.2, 21.6 / 19.8, 28.0 / 24.4, 28.2 / 25.5, of 2048 68.5 / 50.9, 70.8 / 59.7, 93.7 / 74.4, 95.0 / 80.4; 700 of 512 (308)
//     at 33 / 38 38.8 / 34.8, 38.8 / 36.7, of 1024 72.1 / 61.6, 72.5 / 66.0.  Beyond: 768 of 512 (336) 38.8 / 39.8, 38.9 / 41.9; 512 of 1024 (224) x
//     24 37.3 / 40.0; 1000 of 2048 (448) x 24 99.9 / 118.9; fuller: 320 of 1024 (140) x 32 37.8 / 36.4, 700 x 32 53.7 / 55.0.  At 3 to 32 layers 0.77
//     to 0.96 in 42 random launches, with stores in turn and again (1280 channels x 38 at 308 units 1.04 in turn, 0.92 again)
inline int split_tiles(const ScoreArgs& a) {
    constexpr int64_t kSplitUnits = 512, kUnitsOfFourTiles = 256;
    const int64_t units = ((int64_t)a.n_groups + 15) / 16 * a.n_layers;
    const int channels = a.n_kv_heads * a.head_dim;
    const int tiles = (a.t_q + 15) / 16;
    if (units > kSplitUnits) {
        const int64_t wide = ((int64_t)a.n_groups + kGemmN - 1) / kGemmN * a.n_layers;
        if (one_tile_splits(units, wide, a.t_q, channels)) return 1;
        const bool idle = wide <= 168 || (tiles == 3 && wide > 256 && wide <= 308);  // 256 compute units
        return idle && tiles >= 2 && tiles <= 3 && 5 * a.t_q <= 64 * tiles && channels >= 512 ? tiles : 0;
    }
    const int most = units > kUnitsOfFourTiles ? 3 : 4;
    const int passes = (tiles + most - 1) / most;
    return (tiles + passes - 1) / passes;
}

// Groups of a unit of the 64 x 64 form: 64, or 32 where units of 64 need two rounds of the 256 compute units and units of 32 one and a half (257
// units of 64 to 768 of 32). The waves of a unit of 32 share out the token tiles in two halves, so a pass of one or three tiles has an idle one: 17
// to 32 tokens, or more than 48.  Fold and scores, units of 64 / 32, three stores in turn:
//   28 layers x 600 groups of 512 channels (280 units of 64) x 32 tokens 30.2 / 26.7, x 48 39.8 / 40.4, x 64 48.4 / 41.7, x 70 62.0 / 59.5, x 100
//     81.7 / 75.0, x 300 214 / 186; 864 (378) of 64 to 2048 channels x 64 0.84 to 0.91, 620 of 64 x 20 0.96; 164 random launches at 1 to 32 layers,
//     in turn and again, none slower
//   outside the query is staged more often for nothing: 1024 groups (448) x 32 30.4 / 31.7, x 64 49.1 / 55.7; 1300 (588, rounds of 3 and 2.5) 39.5 /
//     37.2, 66.1 / 65.4, x 100 112 / 121; 3600 x 64 141 / 150; up to one round 2 % are gained at 32 and 64, 3 to 4 lost at 100
inline int gemm_width(const ScoreArgs& a) {
    const int64_t units = ((int64_t)a.n_groups + kGemmN - 1) / kGemmN * a.n_layers, halves = ((int64_t)a.n_groups + kGemmN / 2 - 1) / (kGemmN / 2) * a.n_layers;
    const bool pairs = a.t_q > 16 && (a.t_q <= 32 || a.t_q > 48);
    return pairs && units > 256 && halves <= 768 ? kGemmN / 2 : kGemmN;
}

// Tiles of 16 query tokens per pass of score_token_fold_kernel (1 to 4), or 0: the fold is a launch of its own, and split_tiles decides about the
// contraction. What a workgroup has to convert (query heads per KV head x tokens of all passes x channels, twice that in float32) is set against the
// launch that is saved. With the cosine a workgroup also sums what it folded over the tokens; a fold of its own is cut into parts where 64 divides
// the head (`cut`), and takes longer with more workgroups (`fold_blocks`).  Fold and scores alone, us, launch of its own / inside; a number in
// thousands is what the workgroup converts.
//   up to 256 (layer, 16-group) units, one workgroup a compute unit
//     one and two heads, and three and four in 16 bits without the cosine or not `cut`, 600 K: never slower as far as measured (16 on 8 of 256 x 55
//       tokens, 262 K, 41.7 / 34.7)
//     three and four in 16 bits, cosine, `cut`: 16 on 4 of 128 x 123 (262 K) 21 % gained, 24 on 8 of 128 x 91 (295 K) 34.9 / 36.2, 12 on 3 of 256 x
//       98 (393 K) 33.1 / 36.8.  From 1024 channels on: 32 on 8 of 128 x 14 (65 K) 10 % gained, 24 on 8 of 128 x 18 (98 K) 14.0 / 14.4; behind a fold
//       of more than 256 workgroups 32 on 8 of 128 x 60 (262 K) 24 % gained
//     more than four in 16 bits, in turns, 100 K; cosine, `cut`, from 1024 channels on: 40 on 8 of 128 x 9 (82 K) 10.8 / 12.7
//     three and four in float32, in turns: `cut` 8 on 2 of 128 x 49 (131 K) 11.6 / 10.9, 12 on 3 of 128 x 47 (147 K) 12.9 / 13.1, 16 on 4 of 128 x 38
//       (197 K) 13.2 / 15.1, cosine, from 1024 channels on 24 on 8 of 128 x 16 (98 K) 12.0 / 12.7; not `cut` 12 on 3 of 112 x 105 (344 K) 23.2 /
//       18.7, 20 on 5 of 88 x 117 (451 K) 11 % lost, behind a fold of 224 workgroups 24 on 8 of 80 x 119 (492 K) 38.1 / 31.3, of whole blocks of 32
//       channels 32 on 8 of 96 x 26 (197 K) 14.0 / 14.6; behind a fold of 208 workgroups 16 on 4 of 256 x 25 (262 K) 15.9 / 17.6, of 280 15 on 5 of
//       128 x 63 (246 K) 26.9 / 20.9
//     more than four in float32, 100 K: 21 on 3 of 112 x 11 (75 K) 8.8 / 7.2; cosine, `cut`, from 288 channels on 18 on 3 of 128 x 10 (74 K) 8.6 /
//       7.7, 24 on 4 of 128 x 12 (98 K) 9.1 / 9.6; an odd one leaves a turn half empty: 15 on 3 of 128 x 5 (61 K) 8.3 / 7.1, 35 on 5 of 64 x 13 (72
//       K) 8.0 / 8.2
//   257 to 512, two workgroups of at most two tiles a compute unit, three of up to two heads; not where a pass would be partly idle (16 on 4 of 128
//     x 45, in two passes of two, whole question 26.6 / 30.3)
//     up to four heads 270 K; cosine, `cut`, three and four from 768 channels on: 32 on 8 of 128 x 14 (66 K) gained, 12 on 3 of 256 x 20 (98 K)
//       18.6 / 19.2, behind a fold of more than 112 workgroups 32 on 8 of 128 x 22 (131 K) 25.6 / 23.6
//     in turns 60 K; 16 bits, cosine, `cut`: 16 on 2 of 128 x 8 (33 K) 9.3 / 8.1, 12 on 1 of 128 x 28 (49 K) 9.5 / 10.1
//   above, short questions of up to two heads on keys that are not the shortest, whole question: 4 on 4 of 128 x 32, 588 units 27.9 / 21.9, 1064 35.5
//     / 30.0, 1792 35.9 / 38.7; 2 on 2 of 96, 900 20.7 / 19.1; 2 on 1 of 64, 1064 14.4 / 15.6
// Few tokens on long keys: a tile is folded whole however empty it is.  1 token, 32 on 8 of 256 21.3 / 24.1, 16 on 8 of 128 (504 units) 22.3 / 23.3,
// 10 on 5 of 256 17.4 / 17.0; 9 to 11 tokens, cosine, 16 on 8 of 256 15.2 / 16.6 (dot 15.0 / 12.4), 8 on 8 of 256 behind a fold of 896 workgroups
// 19.2 / 16.1.
// Scores that share memory with the query need the separate fold, as above.
inline int fold_tiles(const ScoreArgs& a) {
    const int64_t units = ((int64_t)a.n_groups + 15) / 16 * a.n_layers, channels = (int64_t)a.n_kv_heads * a.head_dim;
    const bool is_f32 = a.q_dtype == TOM_F32, few = units <= 256, most_units = units <= 512;
    const bool cosine = a.sim == TOM_SIM_COSINE, cut = a.head_dim % 64 == 0;
    const int r = a.n_q_heads / a.n_kv_heads, heads = is_f32 ? 2 * r : r;
    if (units > 1100 || channels > 3072) return 0;  // q-bar sums: at most 24 KB of LDS
    if (!most_units && (heads > 2 || a.t_q > 32 || channels < 192)) return 0;
    if (a.t_q < 8 && heads * channels > (few ? 4000 : 2000)) return 0;
    const int most = few ? 4 : heads <= 2 && most_units ? 3 : 2;
    const int tiles = (a.t_q + 15) / 16, passes = (tiles + most - 1) / most, of_pass = (tiles + passes - 1) / passes;
    if (!few && passes * of_pass > tiles) return 0;
    const int64_t converted = heads * channels * 16 * of_pass * passes;
    const int64_t fold_blocks = (int64_t)a.n_layers * a.n_kv_heads * (cut ? a.head_dim / 64 : 1);  // of the launch that is saved
    if (a.t_q < 16 && cosine && channels >= 2048 && fold_blocks <= 512) return 0;
    int64_t most_converted = 600000;
    if (!few) {
        if (r > 4 || (is_f32 && r > 2)) most_converted = cosine && cut && !is_f32 ? 45000 : 60000;
        else most_converted = cosine && cut && r > 2 && channels >= 768 && fold_blocks <= 112 ? 90000 : 270000;
    } else if (is_f32 && r > 2) {
        if (r > 4) most_converted = !cosine || !cut || channels < 288 ? 100000 : r % 2 ? 66000 : 76000;
        else if (a.head_dim % 32 != 0) most_converted = fold_blocks > 210 ? 600000 : 400000;
        else if (fold_blocks > 210) most_converted = 280000;
        else if (cut) most_converted = cosine && channels >= 1024 ? 90000 : 140000;
        else most_converted = 190000;
    } else if (r > 4) {
        most_converted = cosine && cut && channels >= 1024 ? 80000 : 100000;
    } else if (r > 2 && cosine && cut) {
        if (channels >= 1024) most_converted = fold_blocks > 256 ? 270000 : 80000;
        else most_converted = fold_blocks > 112 ? 600000 : 290000;
    }
    if (converted > most_converted) return 0;
    // kept small by the line above
    const uint64_t query_bytes = (uint64_t)a.n_layers * (uint64_t)a.n_q_heads * (uint64_t)a.t_q * (uint64_t)a.head_dim * (is_f32 ? 4u : 2u);
    if (!apart(a.q, query_bytes, a.scores, score_span(a.score_stride, a.n_layers, a.n_groups))) return 0;
    if (a.token_scores && !apart(a.q, query_bytes, a.token_scores, sizeof(float) * (uint64_t)a.n_layers * (uint64_t)a.t_q * (uint64_t)a.n_groups)) return 0;
    return of_pass;
}

// ---- head_dim-axis store: who makes the summary keys ----------------------------------------
constexpr int kTallBlock = 1024;  // threads of a workgroup that walks a tall tile
constexpr int64_t kLowTile = 64 << 10, kTallTile = 128 << 10, kTallTile16Bit = 96 << 10;  // bytes of the input

inline int64_t append_items(const QuantArgs& a) { return (int64_t)a.n_kv_heads * a.n_layers * a.n_frames; }  // K tiles
inline int64_t tile_bytes(const QuantArgs& a, bool is_16_bit) { return (int64_t)a.group_tokens * a.head_dim * (is_16_bit ? 2 : 4); }

// Workgroups per key of the cut form: one per 64 channels while each has a compute unit of its own, which halves the trips at d = 128
// (one bf16 frame of 28 x 4 heads 5.0 against 5.4 us; two frames 8.2 against 7.8), otherwise one.
inline int key_parts(const QuantArgs& a) {
    const int64_t parts = a.head_dim / 64;
    return a.head_dim % 64 == 0 && parts * append_items(a) <= 256 ? (int)parts : 1;
}

// Whether K tiles are cut into chunks like V and the keys come from workgroups of their own (quantize_append_cut_kernel) instead of the workgroups
// that walk the K tiles.  Always where the keys are averaged over another tensor. Otherwise that reads K twice, which pays while the launch is bound
// by the longest chain of one workgroup: not where a walk is one trip of four rows per lane, and up to 384 tiles, 256 with float32 input.  us per
// call in a graph, cut / walk, at 4 heads: 196 x 128 bf16 224 tiles 4.5 / 6.0, 336 5.7 / 6.4, 448 6.9 / 6.9; 256 x 64 float32 224 4.1 / 4.8, 336 5.8
// / 5.5; 50 tokens (one trip) x 8 frames 8.4 / 7.4. Of tiles above 64 KB as far as reading K again costs less than the shorter chains gain.  With
// keys in parts that is by the trips of a walk: cut / 1024 threads at 500 x 128 bf16 10 MB of K 6.2 / 8.2, 14 8.8 / 8.5, 21 12.7 / 11.4; 1000 x 128
// 20 MB 12.5 / 13.9, 29 16.4 / 15.3; 2000 x 128 29 MB 19.0 / 22.9, 41 25.0 / 24.1; float32 196 x 128 11.2 MB 5.1 / 5.2, 12.8 6.5 / 5.4; 500 x 128 14
// MB 7.8 / 8.4, 20 11.0 / 10.0.  A key in one part walks its tile too: 196 x 256 bf16 8.0 MB 6.6 / 6.9, 11.2 7.5 / 7.3; 1000 x 64 10 MB 8.1 / 8.1;
// 400 x 96 9.8 MB 6.8 / 7.1; float32 400 x 64 6.6 MB 4.7 / 4.9, 9.8 5.5 / 5.2.
inline bool cut_append(const QuantArgs& a, bool is_16_bit) {
    if (a.ksum != a.k) return true;
    const int64_t items = append_items(a), tile = tile_bytes(a, is_16_bit);
    if (a.group_tokens <= 4 * (kBlock / (a.head_dim / 8)) || 2 * items > (is_16_bit ? 384 : 256)) return false;
    if (tile <= kLowTile) return true;
    const int64_t trips = (int64_t)a.group_tokens * a.head_dim / (4 * 8 * kBlock);
    return items * tile <= (key_parts(a) > 1 ? 9000000 + 800000 * trips : (int64_t)(is_16_bit ? 10 : 8) << 20);
}

// Threads of the workgroups that walk K tiles otherwise.  With 1024 the chain of a tall tile is a quarter as long, but the last of a few trips is
// often nearly empty.  Above 128 KB of input, 96 KB at 16 bits, and above 64 KB up to 384 tiles.  us per call in a graph, 1024 / 256 threads: 500 x
// 128 bf16 (125 KB) 224 tiles 8.5 / 12.7, 448 14.2 / 15.8, 1344 34.7 / 39.4, 7168 223 / 232; 196 x 256 bf16 (98 KB) 448 12.1 / 13.1, 672 16.3 / 17.2,
// 896 20.1 / 19.7, 7168 177 / 181; 330 x 128 bf16 (82 KB) 384 9.3 / 10.2, 512 12.4 / 12.3; 196 x 128 bf16 (49 KB) 448 7.2 / 7.0, 896 12.4 / 11.2.
// float32 196 x 128 (98 KB) 384 8.6 / 9.2, 512 11.6 / 11.2, 896 18.2 / 16.8; 256 x 128 (128 KB) 336 9.3 / 9.3, 1792 43.3 / 40.1; 500 x 128 448 20.6 /
// 21.6, 3584 203 / 212.
inline int walk_threads(const QuantArgs& a, bool is_16_bit) {
    const int64_t tile = tile_bytes(a, is_16_bit);
    return tile > (is_16_bit ? kTallTile16Bit : kTallTile) || (tile > kLowTile && 2 * append_items(a) <= 384) ? kTallBlock : kBlock;
}

// ---- token-axis store: tiles whose rows the waves hold -------------------------------------
constexpr int kMostRows = 8, kMostRows16Bit = 13;  // rows a lane holds at most

// Rows per lane where `waves` waves hold a tile; a wave covers 64 / lpr token rows of lpr lanes a pass.
inline int rows_per_lane(int lpr, int group_tokens, int waves) {
    const int passes = (group_tokens + 64 / lpr - 1) / (64 / lpr);
    return (passes + waves - 1) / waves;
}

// Waves per tile, or 0: the general form (other head sizes, and where it is the better one).  Eight rows per
// lane, at most four waves (seven of eight rows lose to the general form: 196 rows at d = 128, 16 frames
// 56.1 against 52.5 us, since one workgroup more or less per compute unit is then a third of it).
// Taller tiles take 13 rows, where the registers hold them (16-bit inputs): 48.6 us.  At d = 256 a
// wave covers only two rows a pass and the exchange costs more, so 13 rows are taken wherever at
// most one of them per wave is idle (50 rows: 28.5 us against 29.4 with eight rows and 31.6 in the general
// form) and tiles above 32 passes otherwise stay in the general form (80 rows: 50.6 against 47.0).
inline int row_waves(int lpr, int group_tokens, bool is_16_bit) {
    if (lpr != 8 && lpr != 16 && lpr != 32) return 0;
    const int passes = rows_per_lane(lpr, group_tokens, 1);
    const int few = (passes + kMostRows16Bit - 1) / kMostRows16Bit;
    if (lpr == 32 && is_16_bit && few <= 4 && few * kMostRows16Bit - passes <= few) return few;
    if (passes <= 4 * kMostRows) return (passes + kMostRows - 1) / kMostRows;
    return is_16_bit && lpr < 32 && few <= 4 ? 4 : 0;
}

// The general form: rows that a lane holds between its two sweeps over a tile, at most.
constexpr int kMostHeld = 8, kMostHeld16Bit = 13;

// Rows per lane where `threads` of a workgroup share a tile.
inline int held_rows(int lpr, int group_tokens, int threads) { return (group_tokens + threads / lpr - 1) / (threads / lpr); }

// Threads of the general form where 256 cannot hold the tile, or 0: it is read twice.  As few as hold it: 512 leave two workgroups a compute unit, so
// that one loads while the other packs; 1024 one.  28 layers x 4 heads, us per call, twice / 512 / 1024 / waves that hold the tile (8 of them): bf16
// 196 x 256, 6 frames (215 MB) 54.3 / 44.2 / 49.5 / 49.5, one 15.2 / 10.8 / 10.3 / 12.2; 110 x 256, 16 77.6 / 61.8 / 71.3 / 70.2; 250 x 128, 16 87.2
// / 67.6 / 80.8 / 69.1; float32 196 x 128, 16 114 / 87.5 / 104 / 82.7, two 15.7 / 11.5 / 14.3 / 11.9; 240 x 80 85.5 / 70.4 / 94.7; 196 x 96, one 8.2
// / 7.9 / 8.3; 196 x 256, 8 131 / - / 94.0 / 150; bf16 256 x 256 73.5 / - / 60.9 / 86.
inline int tall_threads(int lpr, int group_tokens, bool is_16_bit) {
    for (int threads : {512, 1024})
        if (held_rows(lpr, group_tokens, threads) <= (is_16_bit ? kMostHeld16Bit : kMostHeld)) return threads;
    return 0;
}

// ---- gather: the prefix rows, and the selection ---------------------------------------------
// All ask about a launch whose sizes (from chunks to head_out_bytes) are filled in.

// Whether the prefix rows can be copied by blocks of the gather's own launch.  As a launch of its
// own the copy costs 1.3 to 4.5 us for 14 rows (0.8 MB at 28 layers), inside the gather nothing
// that can be measured.  Not where a grid dimension would pass 2^32 threads, nor where the source
// overlaps the active buffer: the copy then has to come first.
inline bool prefix_joins_gather(const DequantArgs& a) {
    const int64_t heads = (int64_t)a.n_layers * a.n_kv_heads;
    const uint64_t sys_bytes = (uint64_t)(heads * a.prefix_bytes), out_bytes = (uint64_t)(heads * a.head_out_bytes);
    if ((a.prefix_bytes / 16 + kBlock - 1) / kBlock + (int64_t)a.k_eff * a.chunks >= (1LL << 32) / kBlock) return false;
    for (const void* sys : {a.sys_k, a.sys_v})
        for (const void* out : {a.k_out, a.v_out})
            if (!apart(sys, sys_bytes, out, out_bytes)) return false;
    return true;
}

// Whether the codes are read past the caches: where what a question reads, its codes, pairs and keys, is more than the last-level cache (256 MB)
// keeps for the next one.  (The output is written past the caches anyway, keys of kKeysPastCaches and more are read past them.)  Asked for 4-bit
// codes on the head_dim axis with 16-bit output alone: the narrower loads of float32 output were 7 % slower past the caches, the token axis 2 %.
// Below the line a repeated question loses its hits, above it the lines that are brought in only evict each other.  28 layers x 4 heads x 196 x 128,
// us per question, through / past, the same question again: 40 of 200 groups (140 MB and 11 MB of keys) 94 / 106, 56 (197) 133 / 144, 58 (204) 152 /
// 147, 64 (225) 183 / 162; 40 of 1024 (59 MB of keys) 102 / 119, 48 (169) 151 / 138; 56 of 3593 (keys past the caches) 170 / 181, 60 (211) 199 / 191.
// Three stores in turn: 40 of 200 109 / 106, 56 147 / 143, 64 165 / 161.  All groups of a store are one range without holes, which the cache keeps
// further: 72 of 72 (253) 148 / 172, 80 of 80 (281) 197 / 190.
inline bool gather_past_caches(const DequantArgs& a) {
    const int64_t heads = (int64_t)a.n_layers * a.n_kv_heads;
    const int64_t read = heads * 2 * a.k_eff * ((int64_t)a.tile_items * 4 + a.tile_meta_bytes), keys = heads * a.n_groups * a.head_dim * (int64_t)sizeof(float);
    return read + (keys < kKeysPastCaches ? keys : 0) > (a.k_eff == a.n_groups ? 265000000 : 210000000);
}

// Pieces of 4 KB that a workgroup of dequant_gather_pieces_kernel takes, one behind the pieces of the other XCDs' workgroups.
constexpr int kPieces = 2;
constexpr uint32_t kXcds = 8;

// Pieces of the rows of a head: where not all heads' rows start at the start of a piece, the first one may be a part.
inline int64_t pieces_of_head(const DequantArgs& a) {
    constexpr uint64_t kPieceBytes = kBlock * 16;
    const uint64_t prefix = (uint64_t)a.prefix_bytes;
    const uint64_t starts = (reinterpret_cast<uintptr_t>(a.k_out) + prefix) | (reinterpret_cast<uintptr_t>(a.v_out) + prefix) | (uint64_t)a.head_out_bytes;
    const int64_t part = starts % kPieceBytes ? kBlock - 1 : 0;
    return ((int64_t)a.k_eff * a.tile_items + part + kBlock - 1) / kBlock;
}
// ... and its workgroups.
inline int64_t piece_blocks(const DequantArgs& a) { return (pieces_of_head(a) + kPieces - 1) / kPieces; }

// Whether the gather goes by aligned pieces of its output instead of by tiles (dequant_gather_pieces_kernel).  Large launches on the head_dim axis
// alone: the pieces are written in a better order, but a wave of them has a longer way to its first load, which smaller launches do not hide.  By
// tiles / by pieces, us, at 28 layers, three stores in turn (the same question again).
//   16-bit output from 400 MB on: 196 x 128, 200 MB 47.7 / 49.8 (38.6 / 38.7), 300 70.0 / 69.8 (58.3 / 57.7), 450 106.2 / 105.7 (89.3 / 87.9), 700
//     156.3 / 154.2; 50 x 128 200 49.7 / 50.4 (40.1 / 40.5), 450 104.5 / 102.6 (89.6 / 87.2); 61 x 96 700 167.8 / 162.4; 37 x 256 700 162.3 / 152.2;
//     2-bit codes 196 x 128 450 104.8 / 104.8 (80.4 / 79.6), 61 x 96 112.0 / 107.4 (84.6 / 83.7)
//   not 2-bit codes with bfloat16 pairs: 50 x 128 450 MB 92.7 / 98.9
//   not 4-bit tiles of three passes (513 to 768 items) where a head has fewer than 768 pieces: a tile is one workgroup that loads it whole, and such
//     heads change the window often.  400 to 800 MB, by pieces over by tiles, means of random launches: up to 500 pieces 1.02 (1.04), 768 1.01
//     (1.03), 1000 0.99 (1.01), 1500 1.00 (1.01), above 0.98 (0.99); tiles of two passes 0.96 to 1.00 (0.97 to 1.01), of four and more 0.95 to 1.00
//     (0.96 to 1.01), single launches up to 1.08; 2-bit codes of three 0.99 (1.00)
//   float32 output of 2-bit codes from 300 MB to 1 GB: 196 x 128 400 71.7 / 61.2 (69.6 / 61.1), 700 138 / 110 with bfloat16 pairs, 149 / 152 (130 /
//     109) with float32 ones, 1400 265 / 282 (263 / 217)
//   not float32 output of 4-bit codes: 700 151 / 158
// A tile of one pass or less leaves lanes of its workgroup idle, and the workgroup has nothing to hide its loads behind, hence lines of their own at
// 16-bit output, whatever the codes and pairs.
//   up to 208 items from 30 MB on: 16 x 64 (128 items) 32 MB 12.5 / 7.6 (12.6 / 6.4), 390 147 / 85 (129 / 72); 13 x 128 (208) 32 8.9 / 8.2 (8.6 /
//     6.3), 390 123 / 88 (82 / 78); the worst, 20 x 80 (200) in quant-groups of 16, 32 9.5 / 9.5 (8.9 / 6.8), 150 50.1 / 43.1 (34.8 / 35.6), 300
//     101.6 / 73.8 (68.1 / 69.0); in 2 bits 200 62.8 / 51.2 (45.1 / 43.2), with bfloat16 pairs 45.2 / 40.2 (44.5 / 39.9)
//   up to 256 from 170 MB on; below it the nearly full tiles lose in both columns, 31 x 64 (248) 150 MB 30.6 / 33.0 (29.5 / 33.4), 15 x 128 (240)
//     31.1 / 32.7 (29.7 / 32.8), 16 x 128 (256) 158 31.6 / 32.0 (30.3 / 33.2); above it three stores in turn gain more than the same question again
//     loses: 31 x 64 174 38.6 / 36.6 (33.7 / 36.2), 200 51.2 / 41.4 (38.4 / 41.1), 390 107.5 / 88.3 (72.7 / 78.4), 600 160 / 139 (160 / 139); 16 x
//     128 200 46.2 / 40.8 (37.5 / 39.5), 390 104.6 / 84.1 (71.3 / 72.1)
// Where the codes and pairs of a question nearly fill the last-level cache (185 to 280 MB), the same question again misses more by pieces: 2-bit
// codes with float32 pairs on average 3 % slower at 16 bits and 8 % at float32, single launches up to 20 %, and stores in turn 3 to 5 % faster. The
// pieces take 32-bit offsets, and a wave at most two tiles.
inline bool gather_by_pieces(const DequantArgs& a, bool is_16_bit, uint32_t prefix_blocks) {
    const int64_t items = (int64_t)a.k_eff * a.tile_items, heads = 2 * (int64_t)a.n_layers * a.n_kv_heads, out = heads * items * 16;
    if (a.qaxis == TOM_QAXIS_TOKENS || a.tile_items < 64) return false;
    if (is_16_bit && a.tile_items <= kBlock) {
        if (out < (a.tile_items <= 208 ? 30000000 : 170000000)) return false;
    } else {
        if (is_16_bit ? out < 400000000 || (a.bits == 2 && a.meta_bf16) : out < 300000000 || out > 1000000000 || a.bits != 2) return false;
        const bool three_passes = a.tile_items > 2 * kBlock && a.tile_items <= 3 * kBlock;
        if (is_16_bit && a.bits == 4 && three_passes && pieces_of_head(a) < 768) return false;
    }
    constexpr int64_t kMost = 1LL << 31;
    const int64_t code_tile = (int64_t)a.tile_items * (is_16_bit ? 8 : 4) * a.bits / 8;
    return items < kMost / 16 && a.plane_tiles * code_tile < kMost && a.plane_tiles * a.tile_meta_bytes < kMost && (int64_t)a.n_layers * a.k < kMost / 4 &&
           prefix_blocks < 1u << 23;
}

constexpr int kSelectKeys = 4;  // scores per lane where the gather selects its groups

// Waves of each gather workgroup that select its group from the scores (256 scores each; one or all four), or 0: the indices come from a top-k
// launch.  The launch costs 2.5 to 4 us; selecting delays every round of 2048 workgroups by the 1 to 2 us of the selection, which workgroups of four
// passes hide behind each other's loads and stores, shorter ones do not.  So the most workgroups go by the passes of one.  Question with one query
// token at 28 layers x 4 heads, the gather's own selection over the launch, one and three stores in turn:
//   one wave, 50 and 256 scores
//     one and two passes, 4096: 16 x 128 (one) 16 groups (3584 workgroups) 0.96 to 1.04, 20 (4480) 1.01 to 1.10, 32 (7168) 1.16 to 1.23; 50 x 64
//       (two) 18 1.02 to 1.05, 20 1.07 to 1.11; float32 16 x 128 (two) 18 0.99 to 1.01, 24 1.03 to 1.07
//     three, 5632: 196 x 128 (three, five workgroups a tile) 3 (3360) 0.96, 5 (5600) 1.00, 6 (6720) 1.03
//     four, 8192 (on the token axis, where a lane loads 8 pairs first, five; four 4096): 50 x 128 (four) 18 0.91 to 0.97, 32 0.95 to 1.01, 36 (8064)
//       0.97 to 1.02; float32 32 x 128 (four) 32 0.93, token axis 0.92; token axis 50 x 128 (four) 18 0.94 to 0.97, 20 0.99 to 1.03, 32 1.06 to 1.09,
//       80 x 128 (five) 24 0.93 to 0.98, 32 0.95 to 0.98
//   four waves, 300 to 1000 scores
//     up to three passes, 1152: 16 x 128 4 (896) 0.98 to 0.99, 5 (1120) 1.00 to 1.01, 9 (2016) 1.03 to 1.09; 50 x 64 5 0.98 to 1.04, 6 1.00 to 1.06,
//       9 1.04 to 1.11; 196 x 128 1 (1120) 0.98
//     four, 2048: 50 x 128 9 0.97 to 1.00, token axis 0.95 to 1.01
// The launch reads all scores while it writes: no output may share memory with them.
inline int select_waves(const DequantArgs& a) {
    const int waves = a.n_groups <= 64 * kSelectKeys ? 1 : kBlock / 64;
    const int64_t heads = (int64_t)a.n_layers * a.n_kv_heads;
    auto passes_above = [&](uint32_t n) { return a.chunk_items > n * a.step; };
    const bool many_pairs = a.qaxis == TOM_QAXIS_TOKENS && a.lanes_per_row * 8 == (uint32_t)a.head_dim;  // a lane loads 8 pairs first: a pass more
    const int most = waves > 1 ? (passes_above(3) ? 2048 : 1152)
                               : passes_above(many_pairs ? 4 : 3) ? 8192 : passes_above(2) && !many_pairs ? 5632 : 4096;
    if (a.n_groups > kBlock * kSelectKeys || (int64_t)a.k_eff * a.chunks * 2 * heads > most) return 0;
    const uint64_t score_bytes = score_span(a.score_stride, a.n_layers, a.n_groups);
    const uint64_t out_bytes = (uint64_t)(heads * a.head_out_bytes), idx_bytes = 4u * (uint64_t)a.n_layers * (uint64_t)a.k;
    return apart(a.scores, score_bytes, a.k_out, out_bytes) && apart(a.scores, score_bytes, a.v_out, out_bytes) &&
                   apart(a.scores, score_bytes, a.sel_idx, idx_bytes)
               ? waves
               : 0;
}

}  // namespace oqm
