// Driver for the host-side rules of csrc/oqm_dispatch.h, built for the host with
// -fsanitize=address,undefined by tests/test_sanitizers.py.  Both sides of every limit, and buffers that
// overlap, adjoin or lie apart.  No device is touched: the addresses are fakes.  Exit status 0 = clean.
#include <cstdio>

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
    // the line: 28 * 128 query elements a token, 8 workgroups a layer at 256 groups
    a.scores = reinterpret_cast<float*>(at(1 << 28));
    a.n_layers = 8, a.n_groups = 256, a.score_stride = 256, a.t_q = 26;
    CHECK(fold_slots(a) == 8);
    a.t_q = 27;
    CHECK(fold_slots(a) == 0);
    // one round of the chip: one workgroup per compute unit with a float32 query, two with a 16-bit one and short keys
    a.t_q = 1, a.n_layers = 8;
    for (int dtype : {TOM_F32, TOM_BF16, TOM_F16})
        for (int heads : {1, 2}) {
            a.q_dtype = dtype, a.n_kv_heads = a.n_q_heads = heads;
            auto fused = [&](int groups) {
                a.n_groups = groups, a.score_stride = groups;
                return fold_slots(a) > 0;
            };
            CHECK(fused(256 * 32 / 8));
            CHECK(fused(256 * 32 / 8 + 1) == (dtype != TOM_F32));
            CHECK(fused(512 * 32 / 8) == (dtype != TOM_F32));
            CHECK(fused(512 * 32 / 8 + 1) == (dtype != TOM_F32 && heads == 2));
        }
    a.n_layers = 1, a.n_groups = a.score_stride = 256, a.q_dtype = TOM_BF16;
    a.t_q = 1, a.head_dim = 256, a.n_kv_heads = a.n_q_heads = 16;
    CHECK(fold_slots(a) == 1);
    a.n_kv_heads = a.n_q_heads = 17;                   // no row slot left for the last head
    CHECK(fold_slots(a) == 0);
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
}

int main() {
    fold();
    split();
    if (failures) { std::fprintf(stderr, "%d failures\n", failures); return 2; }
    std::printf("dispatch driver: clean\n");
    return 0;
}
