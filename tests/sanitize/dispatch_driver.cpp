// Driver for the host-side rules of csrc/oqm_dispatch.h, built for the host with
// -fsanitize=address,undefined by tests/test_sanitizers.py.  Both sides of every limit, and buffers that
// overlap, adjoin or lie apart.  No device is touched: the addresses are fakes.  Exit status 0 = clean.
#include <cstdio>
#include <utility>
#include <vector>

#include "oqm_dispatch.h"

using namespace oqm;

static int failures = 0;
#define CHECK(cond)                                                          \
    do {                                                                     \
        if (!(cond)) {                                                       \
            std::fprintf(stderr, "line %d: %s does not hold\n", __LINE__, #cond); \
            ++failures;                                                      \
        }                                                                    \
    } while (0)

static char* at(uint64_t address) { return reinterpret_cast<char*>((uintptr_t)address); }

static void fold() {
    ScoreArgs a{};
    a.n_kv_heads = 4, a.n_q_heads = 28, a.head_dim = 128, a.n_layers = 2, a.t_q = 8, a.n_groups = 100;
    a.score_stride = 112, a.q_dtype = TOM_BF16;
    const uint64_t q_bytes = 2ull * 28 * 8 * 128 * 2, s_bytes = (112 + 100) * 4;
    a.q = at(1 << 20);
    auto slots_with_scores_at = [&](uint64_t address) {
        a.scores = reinterpret_cast<float*>(at(address));
        return fold_slots(a);
    };
    const uint64_t q = 1 << 20;
    CHECK(slots_with_scores_at(1 << 24) == 8);        // 512 threads, 16 lanes per row, 4 heads
    CHECK(slots_with_scores_at(q + q_bytes) == 8);    // adjoining, behind
    CHECK(slots_with_scores_at(q - s_bytes) == 8);    // and in front
    CHECK(slots_with_scores_at(q) == 0);
    CHECK(slots_with_scores_at(q + q_bytes - 4) == 0);
    CHECK(slots_with_scores_at(q - s_bytes + 4) == 0);
    CHECK(slots_with_scores_at(q + q_bytes / 2) == 0);
    a.q_dtype = TOM_F32;                               // twice the bytes
    CHECK(slots_with_scores_at(q + q_bytes) == 0);
    CHECK(slots_with_scores_at(q + 2 * q_bytes) == 8);
    // the line: seven rows a token in eight slots, 8 workgroups a layer at 256 groups
    a.scores = reinterpret_cast<float*>(at(1 << 28));
    a.n_layers = 8, a.n_groups = 256, a.score_stride = 256, a.t_q = 18;
    CHECK(fold_slots(a) == 8);
    a.t_q = 19;
    CHECK(fold_slots(a) == 0);
    a.n_layers = 28;                                   // 224 workgroups: ten rows, nine with a float32 question on keys of more than five pieces
    for (int dtype : {TOM_F32, TOM_BF16, TOM_F16}) {
        a.q_dtype = dtype;
        a.t_q = dtype == TOM_F32 ? 10 : 11;
        CHECK(fold_slots(a) == 8);
        ++a.t_q;
        CHECK(fold_slots(a) == 0);
    }
    // float32 on keys of four pieces: question and keys an XCD reads, 1.8 MB of keys and 115 KB a token or 0.9 MB and 57 KB
    a.q_dtype = TOM_F32, a.head_dim = 64, a.n_q_heads = 16;
    auto past_l2 = [&](int layers, int groups, int t_q) {
        a.n_layers = layers, a.n_groups = a.score_stride = groups, a.t_q = t_q;
        return fold_slots(a) == 0;
    };
    CHECK(!past_l2(28, 512, 20) && past_l2(28, 512, 21) && !past_l2(28, 480, 21));
    CHECK(!past_l2(28, 256, 36) && past_l2(28, 256, 37) && !past_l2(14, 512, 40) && past_l2(14, 512, 41));
    CHECK(!past_l2(56, 256, 10) && past_l2(56, 256, 11) && !past_l2(112, 128, 10) && past_l2(112, 128, 11) && past_l2(1 << 30, 1, 1));
    a.q_dtype = TOM_BF16, a.n_q_heads = 28, a.head_dim = 128, a.n_layers = 28;
    a.n_groups = a.score_stride = 1024, a.t_q = 1, a.q_dtype = TOM_BF16;  // several rounds of the chip
    CHECK(fold_slots(a) == 8);
    a.t_q = 2;
    CHECK(fold_slots(a) == 0);
    // one round of the chip: two workgroups per compute unit, one with a float32 query and a key of more than five pieces; longer keys hide the second
    // round of a 16-bit query
    a.t_q = 1, a.n_layers = 8;
    for (int dtype : {TOM_F32, TOM_BF16, TOM_F16})
        for (int heads : {1, 2, 3}) {
            a.q_dtype = dtype, a.n_kv_heads = a.n_q_heads = heads;
            auto fused = [&](int groups) {
                a.n_groups = groups, a.score_stride = groups;
                return fold_slots(a) > 0;
            };
            CHECK(fused(256 * 32 / 8));
            CHECK(fused(256 * 32 / 8 + 1) == (dtype != TOM_F32 || heads < 3));
            CHECK(fused(512 * 32 / 8) == (dtype != TOM_F32 || heads < 3));
            CHECK(fused(512 * 32 / 8 + 1) == (dtype != TOM_F32 && heads > 1));
        }
    a.q_dtype = TOM_F32, a.n_groups = a.score_stride = 512 * 32 / 8;
    a.head_dim = 64, a.n_kv_heads = a.n_q_heads = 5;   // five pieces
    CHECK(fold_slots(a) > 0);
    a.head_dim = 328, a.n_kv_heads = a.n_q_heads = 1;  // and a rest
    CHECK(fold_slots(a) == 0);
    a.n_layers = 1, a.n_groups = a.score_stride = 256, a.q_dtype = TOM_BF16;
    a.t_q = 1, a.head_dim = 256, a.n_kv_heads = a.n_q_heads = 16;
    CHECK(fold_slots(a) == 1);
    a.n_kv_heads = a.n_q_heads = 17;                   // no row slot left for the last head
    CHECK(fold_slots(a) == 0);
    auto parts = [&](int heads, int d, int layers, int t_q = 1, bool want_tokens = false) {
        a.n_kv_heads = heads, a.head_dim = d, a.n_layers = layers, a.t_q = t_q;
        return fold_parts(a, want_tokens);
    };
    // of 64 channels while 512 workgroups hold them, and above three tokens a slot
    CHECK(parts(4, 256, 32) == 4 && parts(4, 256, 33) == 1 && parts(1, 2048, 16) == 32 && parts(1, 2048, 17) == 1);
    CHECK(parts(4, 256, 33, 48, true) == 1 && parts(4, 256, 33, 49, true) == 4 && parts(4, 256, 33, 49) == 1 && parts(4, 128, 65, 97, true) == 2);
    CHECK(parts(4, 64, 65535) == 1 && parts(1, 96, 1) == 1 && parts(1, 8, 1, 1 << 20, true) == 1 && parts(1, 2048, 1 << 20, 7, true) == 32);
}

static void append() {
    QuantArgs a{};
    char k = 0, other = 0;
    a.k = a.ksum = &k, a.n_kv_heads = 4, a.n_layers = 2, a.head_dim = 128, a.group_tokens = 196;
    for (bool is_16_bit : {false, true}) {
        a.n_frames = is_16_bit ? 24 : 16;             // 384 or 256 tiles of K and V, of at most 64 KB
        a.group_tokens = is_16_bit ? 196 : 128;
        CHECK(cut_append(a, is_16_bit));
        ++a.n_frames;
        CHECK(!cut_append(a, is_16_bit));
        a.ksum = &other;                              // keys of another tensor: at any size
        CHECK(cut_append(a, is_16_bit));
        a.ksum = &k;
    }
    a.n_frames = 1;
    for (int d : {8, 64, 80, 128, 2048}) {            // a walk of one trip is no longer than a chunk
        a.head_dim = d;
        a.group_tokens = 4 * (256 / (d / 8));
        CHECK(!cut_append(a, true));
        ++a.group_tokens;
        CHECK(cut_append(a, true));
    }
    a.n_frames = 16, a.head_dim = 128;                // 128 keys of two parts
    CHECK(key_parts(a) == 2);
    a.n_frames = 17;
    CHECK(key_parts(a) == 1);
    a.n_frames = 1;
    for (int d : {8, 80, 96, 1032}) {
        a.head_dim = d;
        CHECK(key_parts(a) == 1);
    }
    a.head_dim = 192;
    CHECK(key_parts(a) == 3);
    a.head_dim = 2048;
    CHECK(key_parts(a) == 32);
    a.n_layers = 32767, a.n_kv_heads = 1023, a.n_frames = 65535;
    CHECK(key_parts(a) == 1 && !cut_append(a, true));
    // taller tiles: cut by the bytes of K, walked by 1024 threads above 64 KB or 128 KB
    auto form = [&](int d, int G, int items, bool is_16_bit) {
        a.head_dim = d, a.group_tokens = G, a.n_kv_heads = 1, a.n_layers = items, a.n_frames = 1;
        return cut_append(a, is_16_bit) ? 0 : walk_threads(a, is_16_bit);
    };
    CHECK(form(128, 256, 192, true) == 0 && form(128, 256, 193, true) == 256);           // 64 KB
    CHECK(form(128, 257, 128, true) == 0 && form(128, 257, 192, true) == 1024 && form(128, 257, 193, true) == 256);
    CHECK(form(128, 384, 193, true) == 256 && form(128, 385, 193, true) == 1024);        // 96 KB, above 384 tiles
    CHECK(form(128, 385, 1 << 20, true) == 1024 && form(128, 256, 1 << 20, false) == 256 && form(128, 257, 1 << 20, false) == 1024);
    CHECK(form(128, 500, 111, true) == 0 && form(128, 500, 115, true) == 1024);          // two parts a key: 14.6 MB at 7 trips
    CHECK(form(128, 2000, 66, true) == 0 && form(128, 2000, 68, true) == 1024);          // 33.8 MB at 31
    CHECK(form(64, 1000, 81, true) == 0 && form(64, 1000, 82, true) == 1024);            // one part: 10 MiB
    CHECK(form(64, 400, 81, false) == 0 && form(64, 400, 82, false) == 1024);            // 8 MiB with float32 input
    CHECK(form(512, 196, 32, true) == 0 && form(512, 196, 33, true) == 0 && form(512, 196, 53, true) == 1024);
}

static void split() {
    ScoreArgs a{};
    auto tiles = [&](int n_layers, int n_groups, int t_q) {
        a.n_layers = n_layers, a.n_groups = n_groups, a.t_q = t_q;
        return split_tiles(a);
    };
    for (int t_q = 1; t_q <= 1100; ++t_q)
        for (int groups : {1, 256 * 16, 256 * 16 + 1, 512 * 16}) {
            const int m = tiles(1, groups, t_q), all = (t_q + 15) / 16, most = groups > 256 * 16 ? 3 : 4;
            const int passes = (all + m - 1) / m;
            CHECK(m >= 1 && m <= most);
            CHECK(passes == (all + most - 1) / most);   // no more passes than the widest would take
            CHECK(m * passes - all < passes);           // and none with a whole idle tile more than it must have
        }
    CHECK(tiles(8, 1024, 64) == 2 && tiles(8, 1025, 64) == 0);   // 512 and 520 units
    CHECK(tiles(512, 16, 1) == 1 && tiles(513, 16, 1) == 0);
    CHECK(tiles(4, 1024, 64) == 4 && tiles(4, 1024, 65) == 3 && tiles(4, 1024, 1 << 20) == 4);
    CHECK(tiles(65535, 0x7fffffff, 1) == 0);                     // far beyond, no overflow
    // one tile of tokens on keys of 256 channels and more: the most tokens, by units a compute unit
    const struct { int channels, most[8]; } one_tile[] = {{248, {16}}, {256, {16, 8, 0, 7}}, {280, {16, 10, 0, 8}}, {288, {16, 11, 4, 8}}, {320, {16, 14, 5, 9}}, {344, {16, 16, 5, 9}}, {352, {16, 16, 5, 9, 3}}, {400, {16, 16, 6, 10, 4}},
                                                          {512, {16, 16, 7, 11, 6, 0, 0, 0}}, {576, {16, 16, 7, 11, 6, 2, 0, 0}}, {768, {16, 16, 8, 12, 8, 3, 0, 0}}, {1024, {16, 16, 9, 13, 9, 5, 1, 0}},
                                                          {1280, {16, 16, 11, 13, 9, 5, 2, 0}}, {2048, {16, 16, 12, 14, 10, 7, 3, 0}}, {3072, {16, 16, 13, 14, 11, 7, 4, 0}}};
    for (const auto& w : one_tile)
        for (int i = 0; i < 8; ++i)
            for (int units : {i ? 256 * (i + 1) + 1 : 1, 256 * (i + 2)}) {
                a.n_kv_heads = w.channels / 8, a.head_dim = 8;
                for (int t_q = 1; t_q <= 16; ++t_q) CHECK(tiles(1, units * 16, t_q) == (t_q <= w.most[i]));
                CHECK(tiles(units, 16, 1) == (w.most[i == 2 ? 3 : i] > 0));   // one group tile a layer: as many units of 64
            }
    a.n_kv_heads = 2, a.head_dim = 128;
    CHECK(tiles(28, 28 * 16, 17) == 0 && tiles(65535, 0x7fffffff, 1) == 0);
    a.n_kv_heads = 4;                                            // two and three tiles, the last mostly empty: up to 168 units of 64, three from 257 to 308 too
    for (int t_q : {17, 25, 26, 32, 33, 38, 39, 48, 49, 64, 65})
        for (int groups : {6 * 64, 6 * 64 + 1, 9 * 64, 9 * 64 + 1, 11 * 64, 11 * 64 + 1})
            CHECK(tiles(28, groups, t_q) == (t_q >= 33 && t_q <= 38 && (groups <= 6 * 64 || (groups > 9 * 64 && groups <= 11 * 64)) ? 3 : t_q <= 25 && groups <= 6 * 64 ? 2 : 0));
    CHECK(tiles(65535, 0x7fffffff, 17) == 0);
    a.n_kv_heads = 31, a.head_dim = 8;
    CHECK(tiles(28, 58 * 16, 1) == 0 && tiles(28, 6 * 64, 17) == 0);
    a.n_kv_heads = a.head_dim = 0;
    auto width = [&](int n_layers, int n_groups, int t_q) {      // units of 32 groups: more than 256 of 64, at most 768
        a.n_layers = n_layers, a.n_groups = n_groups, a.t_q = t_q;
        return gemm_width(a);
    };
    for (int t_q : {1, 16, 17, 32, 33, 48, 49, 64, 65, 1000}) {
        const bool pairs = t_q > 16 && (t_q <= 32 || t_q > 48);
        CHECK(width(1, 256 * 64, t_q) == 64 && width(1, 256 * 64 + 1, t_q) == (pairs ? 32 : 64) && width(1, 768 * 32, t_q) == (pairs ? 32 : 64) && width(1, 768 * 32 + 1, t_q) == 64);
        CHECK(width(65535, 0x7fffffff, t_q) == 64);
    }

    // the fold inside: layers, groups, query tokens, KV heads, query heads of each, head_dim -> tiles of a pass, or 0
    auto fold = [&](int n_layers, int n_groups, int t_q, int heads, int r, int d, int type = TOM_BF16, int sim = TOM_SIM_DOT) {
        ScoreArgs b{};
        b.n_layers = n_layers, b.n_groups = n_groups, b.t_q = t_q, b.n_kv_heads = heads, b.n_q_heads = heads * r, b.head_dim = d, b.q_dtype = type, b.sim = sim;
        b.score_stride = n_groups;
        const uint64_t bytes = (uint64_t)n_layers * heads * r * t_q * d * (type == TOM_F32 ? 4 : 2);
        const uint64_t out = 1ull << 40;
        b.q = at(out - bytes), b.scores = reinterpret_cast<float*>(at(out)), b.token_scores = reinterpret_cast<float*>(at(1ull << 44));
        const int n = fold_tiles(b);
        b.q = at(out - bytes + 4);
        CHECK(fold_tiles(b) == 0);                               // the scores share memory with the query
        b.q = at((1ull << 44) - bytes);
        CHECK(fold_tiles(b) == n);
        b.q = at((1ull << 44) - bytes + 4);
        CHECK(fold_tiles(b) == 0);
        b.token_scores = nullptr;
        CHECK(fold_tiles(b) == n);
        return n;
    };
    CHECK(fold(1, 256, 16, 4, 7, 128) == 1 && fold(1, 256, 17, 4, 7, 128) == 0 && fold(28, 130, 64, 4, 4, 128) == 4 && fold(28, 100, 65, 5, 2, 256) == 3);
    CHECK(fold(28, 60, 64, 8, 4, 256) == 4 && fold(28, 60, 65, 8, 4, 256) == 0);                      // 524 K and 655 K conversions
    CHECK(fold(28, 256, 32, 4, 4, 128) == 2 && fold(28, 256, 33, 4, 4, 128) == 0 && fold(28, 256, 64, 4, 4, 128) == 2 && fold(28, 256, 45, 4, 2, 128) == 3);
    CHECK(fold(28, 256, 16, 4, 7, 128) == 1 && fold(28, 256, 17, 4, 7, 128) == 0);                    // 57 K and 115 K
    CHECK(fold(28, 100, 7, 8, 4, 256) == 0 && fold(28, 60, 8, 8, 4, 256) == 1 && fold(28, 130, 1, 4, 4, 128) == 1);
    CHECK(fold(28, 300, 32, 4, 2, 128) == 2 && fold(28, 300, 33, 4, 2, 128) == 0 && fold(28, 300, 32, 4, 3, 128) == 0 && fold(28, 300, 32, 1, 1, 128) == 0);
    CHECK(fold(1, 1100 * 16, 16, 4, 1, 128) == 1 && fold(1, 1100 * 16 + 1, 16, 4, 1, 128) == 0);
    CHECK(fold(1, 500, 16, 4, 7, 128, TOM_F32) == 0 && fold(28, 130, 64, 4, 4, 128, TOM_F32) == 4 && fold(28, 256, 32, 4, 1, 128, TOM_F32) == 2);
    auto cosine = [&](int n_layers, int n_groups, int t_q, int heads, int r, int d, int type = TOM_BF16) { return fold(n_layers, n_groups, t_q, heads, r, d, type, TOM_SIM_COSINE); };
    // three and four query heads in float32: heads that the fold of its own cuts or not, and one of many workgroups
    CHECK(fold(1, 100, 17, 4, 4, 128, TOM_F32) == 2 && cosine(1, 100, 33, 3, 4, 128, TOM_F32) == 0 && cosine(1, 100, 16, 8, 3, 128, TOM_F32) == 0 && fold(1, 100, 16, 8, 4, 128, TOM_F32) == 1 && cosine(1, 100, 16, 7, 4, 128, TOM_F32) == 1);
    CHECK(cosine(1, 100, 32, 8, 4, 80, TOM_F32) == 2 && cosine(1, 100, 48, 8, 4, 80, TOM_F32) == 3 && cosine(1, 100, 65, 8, 4, 80, TOM_F32) == 0 && cosine(28, 40, 63, 8, 4, 72, TOM_F32) == 4 && cosine(28, 40, 105, 8, 3, 80, TOM_F32) == 4 && cosine(1, 40, 105, 8, 3, 80, TOM_F32) == 0 && fold(1, 100, 32, 8, 4, 96, TOM_F32) == 0 && fold(1, 100, 32, 7, 4, 96, TOM_F32) == 2);
    CHECK(cosine(22, 40, 61, 5, 3, 128, TOM_F32) == 4 && cosine(21, 40, 61, 5, 3, 128, TOM_F32) == 0);
    // more than four in float32
    CHECK(cosine(1, 100, 12, 3, 6, 128, TOM_F32) == 1 && cosine(1, 100, 12, 5, 5, 64, TOM_F32) == 1 && cosine(1, 100, 12, 4, 6, 128, TOM_F32) == 0 && cosine(1, 100, 16, 5, 7, 64, TOM_F32) == 0 && fold(1, 100, 16, 5, 7, 64, TOM_F32) == 1 && cosine(1, 100, 32, 3, 7, 64, TOM_F32) == 2 && cosine(1, 100, 11, 3, 7, 112, TOM_F32) == 1 &&
          cosine(1, 100, 17, 3, 7, 96, TOM_F32) == 0);
    // 16 bits with the cosine
    CHECK(cosine(1, 100, 144, 4, 4, 128) == 0 && fold(1, 100, 144, 4, 4, 128) == 3 && cosine(1, 100, 128, 4, 4, 128) == 4 && cosine(28, 100, 145, 4, 4, 128) == 4);
    CHECK(cosine(1, 100, 16, 8, 4, 128) == 1 && cosine(1, 100, 17, 8, 4, 128) == 0 && cosine(28, 60, 64, 8, 4, 128) == 4 && cosine(28, 60, 65, 8, 4, 128) == 0 && cosine(1, 100, 17, 8, 4, 136) == 2);
    CHECK(cosine(1, 100, 9, 8, 5, 128) == 0 && fold(1, 100, 9, 8, 5, 128) == 1 && cosine(1, 100, 9, 7, 5, 128) == 1);
    CHECK(cosine(1, 4100, 17, 4, 4, 128) == 2 && cosine(1, 4100, 17, 3, 4, 256) == 0 && cosine(10, 410, 17, 3, 4, 256) == 2 && cosine(1, 4100, 17, 1, 12, 128) == 0 && cosine(1, 4100, 16, 1, 12, 128) == 1);
    // a tile that is partly empty on the longest keys
    CHECK(cosine(1, 100, 15, 8, 1, 256) == 0 && cosine(1, 100, 16, 8, 1, 256) == 1 && fold(1, 100, 15, 8, 1, 256) == 1 && cosine(1, 100, 15, 8, 1, 248) == 1 && cosine(17, 100, 15, 8, 1, 256) == 1 && cosine(16, 100, 15, 8, 1, 256) == 0);
    // the launches that ask the split form itself (tests/test_gpu_token_split.py): the scores start where the question does
    auto split_alone = [&](int n_layers, int n_groups, int t_q, int heads, int r, int d) {
        ScoreArgs b{};
        b.n_layers = n_layers, b.n_groups = n_groups, b.t_q = t_q, b.n_kv_heads = heads, b.n_q_heads = heads * r, b.head_dim = d, b.q_dtype = TOM_BF16;
        b.score_stride = n_groups + 3, b.q = at(1 << 20), b.scores = reinterpret_cast<float*>(at(1 << 20)), b.token_scores = reinterpret_cast<float*>(at(1ull << 44));
        CHECK(fold_tiles(b) == 0);
        b.sim = TOM_SIM_COSINE;
        CHECK(fold_tiles(b) == 0);
        return split_tiles(b);
    };
    const int channels[][2] = {{1, 8}, {3, 8}, {1, 72}, {1, 128}, {17, 8}, {33, 8}, {65, 8}};
    const int tokens[][2] = {{1, 1}, {16, 1}, {17, 2}, {33, 3}, {48, 3}, {49, 4}, {64, 4}, {65, 3}, {113, 4}, {130, 3}};   // tiles of a pass: 1, 2, 3, 4, 2 x 3, 2 x 4, 3 x 3
    for (const auto& c : channels)
        for (const auto& t : tokens)
            for (int groups : {1, 15, 16, 17})
                for (int r : {1, 2}) CHECK(split_alone(2, groups, t[0], c[0], r, c[1]) == t[1]);
    const int shapes[][3] = {{1, 24, 3}, {1, 40, 33}, {3, 8, 49}, {5, 24, 64}, {1, 24, 97}};
    const struct { int layers, groups, tiles[5]; } launches[] = {{1, 4096, {1, 3, 4, 4, 4}}, {1, 4097, {1, 3, 2, 2, 3}}, {16, 512, {1, 3, 2, 2, 3}}, {16, 513, {}}, {1, 8191, {1, 3, 2, 2, 3}}, {3, 2720, {1, 3, 2, 2, 3}}, {3, 2721, {}}};
    for (const auto& l : launches)
        for (int i = 0; i < 5; ++i) CHECK(split_alone(l.layers, l.groups, shapes[i][2], shapes[i][0], 1, shapes[i][1]) == l.tiles[i]);
    for (int groups : {9600, 9601}) {
        CHECK(split_alone(1, groups, 8, 1, 3, 264) == 1 && split_alone(1, groups, 9, 1, 3, 264) == 0 && split_alone(1, groups, 16, 65, 3, 8) == 1 && split_alone(1, groups, 20, 65, 3, 8) == 2 && split_alone(1, groups, 26, 65, 3, 8) == 0 &&
              split_alone(1, groups, 36, 65, 3, 8) == 3);
        CHECK(fold(1, groups, 8, 1, 3, 264) == 0 && fold(1, groups, 16, 65, 3, 8) == 0);   // apart from the question too
    }
    CHECK(fold(1, 16, 8, 48, 1, 64) == 1 && fold(1, 16, 8, 49, 1, 64) == 0 && fold(65535, 1 << 26, 1 << 20, 1, 1, 8) == 0);
}

static void rows() {
    // lanes per row, 16-bit input, rows of a tile -> waves (0: general form), rows per lane
    const struct { int lpr; bool narrow; int tokens, waves, rows; } want[] = {
        {16, true, 1, 1, 1},    {16, true, 32, 1, 8},   {16, true, 33, 2, 5},   {16, true, 50, 2, 7},   {16, true, 96, 3, 8},
        {16, true, 97, 4, 7},   {16, true, 128, 4, 8},  {16, true, 129, 4, 9},  {16, true, 208, 4, 13}, {16, true, 209, 0, 0},
        {16, false, 128, 4, 8}, {16, false, 129, 0, 0}, {8, true, 64, 1, 8},    {8, true, 65, 2, 5},    {8, true, 256, 4, 8},
        {8, true, 416, 4, 13},  {8, true, 417, 0, 0},   {8, false, 257, 0, 0},  {32, true, 26, 1, 13},  {32, true, 24, 1, 12},
        {32, true, 22, 2, 6},   {32, true, 50, 2, 13},  {32, true, 64, 4, 8},   {32, true, 65, 0, 0},   {32, true, 72, 3, 12},
        {32, true, 104, 4, 13}, {32, true, 105, 0, 0},  {32, false, 26, 2, 7},  {32, false, 64, 4, 8},  {32, false, 65, 0, 0},
        {12, true, 16, 0, 0},   {10, true, 50, 0, 0},   {1, true, 16, 0, 0},    {64, true, 16, 0, 0},   {512, false, 1, 0, 0},
    };
    for (const auto& w : want) {
        const int waves = row_waves(w.lpr, w.tokens, w.narrow);
        CHECK(waves == w.waves);
        CHECK(!waves || rows_per_lane(w.lpr, w.tokens, waves) == w.rows);
    }
    for (int lpr : {8, 16, 32})
        for (bool narrow : {false, true})
            for (int tokens = 1; tokens < 3000; ++tokens) {
                const int waves = row_waves(lpr, tokens, narrow);
                CHECK(waves >= 0 && waves <= 4);
                if (!waves) continue;
                const int held = rows_per_lane(lpr, tokens, waves);
                CHECK(held <= (narrow ? kMostRows16Bit : kMostRows));
                CHECK(waves * held * (64 / lpr) >= tokens);   // every row has a lane
            }
}

static void tall() {
    // 512 threads hold 13 rows a lane at 16 bits, eight of float32, then 1024; a taller tile is read twice
    for (int lpr : {10, 12, 16, 32, 64, 256})
        for (bool narrow : {false, true}) {
            const int most = narrow ? kMostHeld16Bit : kMostHeld;
            CHECK(tall_threads(lpr, most * (512 / lpr), narrow) == 512 && tall_threads(lpr, most * (512 / lpr) + 1, narrow) == 1024);
            CHECK(tall_threads(lpr, most * (1024 / lpr), narrow) == 1024 && tall_threads(lpr, most * (1024 / lpr) + 1, narrow) == 0);
            for (int tokens = 1; tokens < 2000; ++tokens)
                if (const int threads = tall_threads(lpr, tokens, narrow)) CHECK(held_rows(lpr, tokens, threads) * (threads / lpr) >= tokens);
        }
}

static void gather() {
    DequantArgs a{};
    a.n_kv_heads = 4, a.head_dim = 64, a.n_layers = 2, a.k = 10, a.k_eff = 10, a.n_groups = 200, a.chunks = 1;
    a.score_stride = 208, a.prefix_bytes = 5 * 64 * 2, a.head_out_bytes = a.prefix_bytes + 10 * 16 * 64 * 2;
    const uint64_t sys_bytes = 8 * a.prefix_bytes, out_bytes = 8 * a.head_out_bytes, s_bytes = (208 + 200) * 4;
    const uint64_t k_out = 1 << 24, v_out = 1 << 25, idx = 1 << 20, far = 1 << 28, idx_bytes = 2 * 10 * 4;
    a.k_out = at(k_out), a.v_out = at(v_out), a.sel_idx = reinterpret_cast<int32_t*>(at(idx));
    auto scores_at = [&](uint64_t address) {
        a.scores = reinterpret_cast<float*>(at(address));
        return select_waves(a);
    };
    CHECK(scores_at(far) == 1);
    for (const auto& [begin, bytes] : {std::pair<uint64_t, uint64_t>{k_out, out_bytes}, {v_out, out_bytes}, {idx, idx_bytes}}) {
        CHECK(scores_at(begin + bytes) == 1);       // adjoining, behind
        CHECK(scores_at(begin - s_bytes) == 1);     // and in front
        CHECK(scores_at(begin + bytes - 4) == 0);
        CHECK(scores_at(begin - s_bytes + 4) == 0);
        CHECK(scores_at(begin) == 0);
    }
    a.scores = reinterpret_cast<float*>(at(far));
    // one wave for up to 256 scores and 4096 workgroups, 5632 of three passes, 8192 of four (five where every lane loads the pairs of 8 channels); four
    // for up to 1024 scores and 1152 workgroups, 2048 of four passes
    auto waves = [&](int n_groups, int k, int chunks, int passes = 1) {
        a.n_groups = n_groups, a.k = a.k_eff = k, a.chunks = (uint32_t)chunks, a.n_layers = 1, a.n_kv_heads = 1;
        a.step = 256, a.chunk_items = (uint32_t)passes * 256 - 255;
        return select_waves(a);
    };
    for (int axis : {TOM_QAXIS_HEAD_DIM, TOM_QAXIS_TOKENS})
        for (int channels : {4, 8})
            for (int passes : {1, 2, 3, 4, 5}) {
                a.qaxis = axis, a.lanes_per_row = 64 / (uint32_t)channels;
                const bool pairs = axis == TOM_QAXIS_TOKENS && channels == 8;
                const int one = passes > (pairs ? 4 : 3) ? 64 : passes == 3 && !pairs ? 44 : 32, four = passes > 3 ? 16 : 9;
                CHECK(waves(256, 64, one, passes) == 1 && waves(256, 65, one, passes) == 0);
                CHECK(waves(257, 64, four, passes) == 4 && waves(257, 65, four, passes) == 0);
                CHECK(waves(1024, 64, four, passes) == 4 && waves(1024, 65, four, passes) == 0);
            }
    CHECK(waves(256, 255, 4) == 1 && waves(1025, 1, 1) == 0 && waves(1 << 30, 1, 1) == 0);

    // codes, pairs and keys of the question against what the last-level cache keeps; keys of 100 MB and more are not kept
    auto past = [&](int k_eff, int n_groups, int n_layers = 28) {
        DequantArgs q{};
        q.n_layers = n_layers, q.n_kv_heads = 4, q.head_dim = 128, q.k = q.k_eff = k_eff, q.n_groups = n_groups;
        q.tile_items = 196 * 16, q.tile_meta_bytes = 196 * 2 * 8;
        return gather_past_caches(q);
    };
    CHECK(!past(56, 200) && past(58, 200) && !past(40, 1024) && past(48, 1024) && !past(59, 3600) && past(60, 3600));
    CHECK(!past(64, 64) && past(64, 65 + 135) && !past(72, 72) && past(80, 80) && !past(64, 1024, 7) && past(256, 1024, 7));

    // 400 MB of 16-bit output; with float32 output 2-bit codes between 300 MB and 1 GB.  39 groups of 196 x 128: 438 MB
    auto pieces = [&](int64_t k_eff, bool is_16_bit, int bits, bool meta_bf16 = false, int n_layers = 28, int tokens = 196, int capacity = 1024, int k = 0, uint32_t prefix_blocks = 0) {
        DequantArgs q{};
        q.n_layers = n_layers, q.n_kv_heads = 4, q.head_dim = 128, q.k_eff = (int32_t)k_eff, q.k = k ? k : (int32_t)k_eff, q.bits = bits, q.meta_bf16 = meta_bf16;
        q.tile_items = (uint32_t)tokens * (is_16_bit ? 16u : 32u), q.tile_meta_bytes = (uint32_t)tokens * 2 * 8, q.plane_tiles = (int64_t)capacity * 4;
        q.qaxis = TOM_QAXIS_HEAD_DIM;
        const bool yes = gather_by_pieces(q, is_16_bit, prefix_blocks);
        q.qaxis = TOM_QAXIS_TOKENS;
        CHECK(!gather_by_pieces(q, is_16_bit, prefix_blocks));
        return yes;
    };
    CHECK(!pieces(39, true, 4, false, 25) && pieces(39, true, 4, false, 26) && pieces(39, true, 4, true) && pieces(39, true, 2) && !pieces(39, true, 2, true));
    for (int k = 36; k < 129; ++k) CHECK(pieces(k, true, 4));                                  // whatever the last round of a head is left with
    CHECK(!pieces(39, false, 2, false, 9) && pieces(39, false, 2, true, 10) && pieces(39, false, 2, false, 31) && !pieces(39, false, 2, false, 32) && !pieces(39, false, 4, false, 20));
    CHECK(pieces(3000, true, 4, false, 28, 4) && !pieces(3000, true, 4, false, 28, 3));        // 64 items: a wave meets two tiles at most
    CHECK(pieces(39, true, 4, false, 28, 196, 42000) && !pieces(39, true, 4, false, 28, 196, 43000));   // codes of a (layer, K|V) against 2^31 bytes
    CHECK(!pieces(42800, true, 4) && pieces(42700, true, 4));                                  // rows of a head
    CHECK(!pieces(39, true, 4, false, 28, 196, 1024, 1 << 25) && !pieces(39, true, 4, false, 28, 196, 1024, 0, 1u << 23));
    // tiles of up to one pass: 208 items from 30 MB up, 256 from 170
    CHECK(pieces(41, true, 2, true, 28, 13) && !pieces(40, true, 4, false, 28, 13) && pieces(186, true, 4, false, 28, 16) && !pieces(185, true, 4, false, 28, 16) && !pieces(186, true, 4, false, 28, 17));
    // 4-bit tiles of three passes: heads of 768 pieces and more
    for (int tokens : {33, 48})
        CHECK(!pieces(196351 / (tokens * 16), true, 4, false, 21, tokens) && pieces(196353 / (tokens * 16) + 1, true, 4, false, 21, tokens) && pieces(196351 / (tokens * 16), true, 2, false, 21, tokens));
    CHECK(pieces(383, true, 4, false, 21, 32) && pieces(250, true, 4, false, 21, 49));
    // the first piece is a part where the rows of some head do not start on a piece
    DequantArgs starts{};
    starts.k_eff = 64, starts.tile_items = 196 * 16, starts.head_out_bytes = 64 * 196 * 256;
    CHECK(pieces_of_head(starts) == 784 && piece_blocks(starts) == 392);
    starts.k_out = at(1 << 24), starts.v_out = at((1 << 25) + 16);
    CHECK(pieces_of_head(starts) == 785 && piece_blocks(starts) == 393);
    starts.prefix_bytes = 4080;
    CHECK(pieces_of_head(starts) == 785);
    starts.k_out = at((1 << 24) + 16);
    CHECK(pieces_of_head(starts) == 784);
    starts.head_out_bytes += 16;
    CHECK(pieces_of_head(starts) == 785);
    // 64 groups behind 14 prefix rows, and in buffers that start 512 bytes behind a piece, as without either
    DequantArgs behind{};
    behind.n_layers = 28, behind.n_kv_heads = 4, behind.head_dim = 128, behind.k_eff = behind.k = 64, behind.bits = 4, behind.qaxis = TOM_QAXIS_HEAD_DIM;
    behind.tile_items = 196 * 16, behind.tile_meta_bytes = 196 * 2 * 8, behind.plane_tiles = 1024 * 4;
    behind.k_out = at(1 << 24), behind.v_out = at(1ull << 40);
    for (int rows : {0, 1, 14, 16}) {
        behind.prefix_bytes = rows * 256, behind.head_out_bytes = behind.prefix_bytes + 64 * 196 * 256;
        for (int off : {0, 512}) {
            behind.k_out = at((1 << 24) + off);
            CHECK(gather_by_pieces(behind, true, 1));
        }
    }
    // every piece of a head is taken once: rounds of 16 pieces by eight workgroups, the last one by what is left of them
    for (int items : {1, 255, 256, 257, 784 * 256, 785 * 256, 13 * 256 + 1})
        for (int more = 0; more < 40; ++more) {
            starts = DequantArgs{};
            starts.k_eff = 1, starts.tile_items = (uint32_t)(items + more * 256);
            const int blocks = (int)piece_blocks(starts), pieces = (int)pieces_of_head(starts);
            std::vector<int> taken(pieces + 1);
            for (int x = 0; x < blocks; ++x) {
                const int round = x & ~7, apart = blocks - round < 8 ? blocks - round : 8;
                for (int q = 0; q < kPieces; ++q) {
                    const int at_piece = round * kPieces + (x & 7) + q * apart;
                    if (at_piece <= pieces) ++taken[at_piece];
                    CHECK(at_piece <= pieces);
                }
            }
            for (int q = 0; q < pieces; ++q) CHECK(taken[q] == 1);
            CHECK(taken[pieces] == (pieces & 1));
        }

    auto joins = [&](uint64_t sys_k, uint64_t sys_v) {
        a.n_layers = 2, a.n_kv_heads = 4;
        a.sys_k = at(sys_k), a.sys_v = at(sys_v);
        return prefix_joins_gather(a);
    };
    CHECK(joins(far, far + sys_bytes) && joins(far, far));
    for (uint64_t out : {k_out, v_out}) {
        CHECK(joins(out + out_bytes, far) && joins(far, out - sys_bytes));
        CHECK(!joins(out + out_bytes - 16, far) && !joins(far, out + out_bytes - 16));
        CHECK(!joins(out - sys_bytes + 16, far) && !joins(far, out - sys_bytes + 16));
        CHECK(!joins(out, far) && !joins(far, out));
    }
    a.chunks = 1, a.k = a.k_eff = (1 << 24) - 4;    // three blocks of prefix and 2^24 - 4 of the gather; 2^24 x 256 threads are too many
    a.prefix_bytes = 3 * 256 * 16, a.head_out_bytes = 0;
    CHECK(joins(far, far));
    ++a.k_eff;
    CHECK(!joins(far, far));
}

int main() {
    fold();
    append();
    split();
    rows();
    tall();
    gather();
    if (failures) { std::fprintf(stderr, "%d failures\n", failures); return 2; }
    std::printf("dispatch driver: clean\n");
    return 0;
}
