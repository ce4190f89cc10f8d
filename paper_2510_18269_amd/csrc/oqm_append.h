// What the store kernels of both quantization axes share: their arguments and the place of a tile.
#pragma once

#include "oqm_common.h"
#include "oqm_device.h"

namespace oqm {

// What the kernels need of a QuantArgs, made on the host: offsets in bytes, and the constants their divisions and products take.
struct AppendArgs {
    const char *k, *v, *ksum;
    uint64_t frame_bytes, layer_bytes, head_bytes;  // strides of the inputs
    char *codes, *meta, *keys;                      // of the first layer and the first appended group
    uint64_t plane_tiles, key_plane_bytes;          // tiles of a (layer, K|V), bytes of a layer's keys
    uint32_t row_bytes, tile_code_bytes, tile_meta_bytes, key_bytes;
    uint32_t heads, layers, items;                  // items: (frame, layer, head), head fastest, the order of a contiguous input
    int32_t tokens, rows_per_pass, chunks, chunk_rows;
    uint32_t lanes_per_row, inv_lanes_per_row, inv_heads, inv_layers, inv_chunks;
    uint32_t key_parts, inv_key_parts;  // quantize_append_cut_kernel: workgroups per key
    uint32_t first_block;               // of this launch
};

// All but items, rows_per_pass and what follows from them.
inline AppendArgs append_args(const QuantArgs& q, uint32_t elem_bytes, uint32_t pairs_per_tile) {
    AppendArgs a{};
    a.k = static_cast<const char*>(q.k);
    a.v = static_cast<const char*>(q.v);
    a.ksum = static_cast<const char*>(q.ksum);
    a.frame_bytes = (uint64_t)q.stride_frame * elem_bytes;
    a.layer_bytes = (uint64_t)q.stride_layer * elem_bytes;
    a.head_bytes = (uint64_t)q.stride_head * elem_bytes;
    a.row_bytes = (uint32_t)q.stride_token * elem_bytes;  // a tile spans less than 2 GiB
    a.tokens = q.group_tokens;
    a.lanes_per_row = (uint32_t)q.head_dim / 8u;
    a.tile_code_bytes = (uint32_t)q.group_tokens * a.lanes_per_row * (uint32_t)q.bits;
    a.tile_meta_bytes = pairs_per_tile * (q.meta_bf16 ? 4u : 8u);
    a.key_bytes = (uint32_t)q.head_dim * sizeof(float);
    a.plane_tiles = (uint64_t)q.capacity_groups * q.n_kv_heads;
    a.key_plane_bytes = a.plane_tiles * a.key_bytes;
    const uint64_t before = (uint64_t)q.first_group * q.n_kv_heads;  // tiles of a plane in front of the appended ones
    a.codes = reinterpret_cast<char*>(q.codes) + (2u * q.layer0 * a.plane_tiles + before) * a.tile_code_bytes;
    a.meta = static_cast<char*>(q.meta) + (2u * q.layer0 * a.plane_tiles + before) * a.tile_meta_bytes;
    a.keys = reinterpret_cast<char*>(q.keys) + q.layer0 * a.key_plane_bytes + before * a.key_bytes;
    a.heads = (uint32_t)q.n_kv_heads;
    a.layers = (uint32_t)q.n_layers;
    a.inv_lanes_per_row = reciprocal_u32(a.lanes_per_row);
    a.inv_heads = reciprocal_u32(a.heads);
    a.inv_layers = reciprocal_u32(a.layers);
    return a;
}

// Launches `blocks` workgroups of a 1-D grid: at once, except for millions of them, since a grid stays below 2^32 threads.
template <typename GO>
inline hipError_t launch_blocks(AppendArgs& a, int64_t blocks, int threads, GO go) {
    const int64_t most = ((1LL << 32) - 1) / threads;
    for (int64_t b = 0; b < blocks; b += most) {
        a.first_block = (uint32_t)b;
        go(dim3((unsigned)(blocks - b < most ? blocks - b : most)), dim3(threads));
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

// Requests the arguments of the address arithmetic in one go: the compiler would load them where they are
// used, one round trip through the scalar cache after the other.
__device__ __forceinline__ void request(const AppendArgs& a) {
    asm volatile("" ::"s"(a.k), "s"(a.v), "s"(a.frame_bytes), "s"(a.layer_bytes), "s"(a.head_bytes), "s"(a.codes), "s"(a.meta),
                 "s"(a.plane_tiles), "s"(a.row_bytes), "s"(a.tile_code_bytes), "s"(a.tile_meta_bytes), "s"(a.heads), "s"(a.layers),
                 "s"(a.items), "s"(a.tokens), "s"(a.lanes_per_row), "s"(a.inv_heads), "s"(a.inv_layers), "s"(a.keys),
                 "s"(a.key_plane_bytes), "s"(a.key_bytes));
}

struct Item {
    uint32_t f, li, h;
    __device__ __forceinline__ Item(const AppendArgs& a, uint32_t item) {
        const uint32_t fl = div_by(item, a.heads, a.inv_heads);
        h = item - fl * a.heads;
        f = div_by(fl, a.layers, a.inv_layers);
        li = fl - f * a.layers;
    }
    __device__ __forceinline__ uint64_t input(const AppendArgs& a) const {
        return f * a.frame_bytes + li * a.layer_bytes + h * a.head_bytes;
    }
    __device__ __forceinline__ float* key(const AppendArgs& a) const {
        return reinterpret_cast<float*>(a.keys + li * a.key_plane_bytes + (uint64_t)(f * a.heads + h) * a.key_bytes);
    }
};

// Where a tile is stored.
template <bool MB>
struct Stored {
    char* codes;
    typename MetaPair<MB>::type* meta;  // two float32, or two bfloat16 in one word
    __device__ __forceinline__ Stored(const AppendArgs& a, const Item& t, uint32_t kv) {
        const uint64_t tile = (t.li * 2u + kv) * a.plane_tiles + (t.f * a.heads + t.h);
        codes = a.codes + tile * a.tile_code_bytes;
        meta = reinterpret_cast<typename MetaPair<MB>::type*>(a.meta + tile * a.tile_meta_bytes);
    }
};

}  // namespace oqm
