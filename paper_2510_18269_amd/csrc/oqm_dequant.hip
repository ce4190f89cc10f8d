// Reconstruction of the selected frame-groups into the bounded active KV buffer
// (paper Sec. 3.4, Eq. 11 and Eq. 13; supplement "Cache reconstruction for decoding").
//
// dequant_gather_kernel, by tiles: grid (rank * chunks + chunk, then prefix blocks; K|V * H_k + head; layer).  A workgroup of 256
// threads owns one head tile of one selected group where few passes cover it, otherwise an equal share of
// it (launch_t); consecutive workgroups
// write consecutive row blocks of the active buffer.  It reads the group index from device memory
// (the index array never visits the host), streams its rows' packed codes and (scale, zero) pairs,
// and writes them to token rows [rank*G, (rank+1)*G) of the layer's active buffer.  A lane turns the codes of
// 16 bytes of output (8 channels, 4 in float32) into one 128-bit non-temporal store, so each store
// instruction of a wave writes 1 KB of contiguous memory.  HBM-bound: 0.5 + 8/gs bytes
// read and 2 bytes written per element.  It serves the token axis, every launch that selects its groups itself, and those of the head_dim axis
// below the lines of gather_by_pieces (oqm_dispatch.h); above them dequant_gather_pieces_kernel cuts the output into pieces instead.
//
// What its form was chosen by, measured at 28 layers x 64 random groups x 196 x 128 (944 MB), which goes by pieces now (156 us): 163 us
// (5.8 TB/s) in a kernel trace on the fastest card seen and 169 (5.6) on another, where an
// arithmetic-free linear stream of the same byte mix reaches 6.1 TB/s.  Before the stores stopped waiting for each other (below) a
// workgroup lived 3.5 us (index 0.2, loads 1.5, stores 1.7) and 1520 of 2048 slots were taken at any time; one to
// five passes per workgroup, 256 or 512 threads and a barrier between loads and stores
// all stayed within 1 %; seven passes 171, 1024 threads 165, three or five workgroups per compute unit
// instead of eight 230 / 181, and a persistent loop that loads the next piece before it
// stores the current one 187 us: the memory system prefers workgroups whose reads and writes
// are separate bursts.  All heads' K before all heads' V (162 us) is 1 % faster than K and V of a
// head in turn; contiguous instead of random groups take 156 us.
#include <type_traits>

#include "oqm_common.h"
#include "oqm_device.h"
#include "oqm_dispatch.h"
#include "oqm_select.h"

namespace oqm {
namespace {

// System-token prefix (the part of the paper's dual-structure memory that stays in 16 bits): piece
// `block` (256 lanes x 16 bytes) of the prefix rows of one head's active buffer, bit for bit.
__device__ __forceinline__ void copy_prefix(const char* src, char* dst, int64_t bytes, unsigned block) {
    const int64_t off = ((int64_t)block * kBlock + threadIdx.x) * 16;
    if (off < bytes) *reinterpret_cast<u32x4*>(dst + off) = *reinterpret_cast<const u32x4*>(src + off);
}

// The items of a tile (N channels: 16 bytes of output, so that a store of a wave writes 1 KB) are numbered row by row: item
// row * (d/N) + slot.  Codes and output are linear in that number, and so are the pairs of the
// head_dim axis (d/N is a multiple of the gs/N lanes of a quant-group), so a chunk is a linear stream and the
// kernel divides by nothing.  On the token axis a lane has to keep its channels: its items are
// `step` = the largest multiple of d/N below 256 apart, otherwise 256.
// With float32 output, items of 8 channels are two stores of every other 16 bytes each: 28 layers x 20 groups x 4 x 196 x 128 (549 MB)
// 177 us past the caches and 142 through them, items of 4 channels 98 (5.6 TB/s); token axis 185, 145 and 82. (8 channels stay where a
// row of d/4 lanes does not fit the workgroup.)
// kUnroll: items per lane; all their loads are issued before the first is converted, and the host
// cuts the tile into chunks that one trip covers.
// SELECT: waves of the workgroup that select its group from the layer's scores (256 scores each), or 0: the
// index comes from memory; kPastCaches: the same, and the codes are read past the caches (gather_past_caches in oqm_dispatch.h).
constexpr int kPastCaches = -1;

template <typename OUT, int N, int kUnroll, bool TOKEN_AXIS, int BITS, bool MB, int SELECT>
__global__ void __launch_bounds__(kBlock) dequant_gather_kernel(const DequantArgs a) {
    constexpr int EB = elem_bytes<OUT>::value;
    constexpr uint32_t CW = BITS * N / 8;  // bytes of packed codes per item
    constexpr uint32_t CMASK = (1u << BITS) - 1u;
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    const uint32_t tid = threadIdx.x;
    // everything the addresses need is requested at once, not behind the index
    asm volatile("" ::"s"(a.codes), "s"(a.meta), "s"(a.plane_tiles), "s"(a.tile_meta_bytes), "s"(a.tile_items), "s"(a.step),
                 "s"(a.prefix_bytes), "s"(a.head_out_bytes), "s"(a.chunk_items), "s"(a.layer0), "s"(a.lpg_shift), "s"(a.k_out),
                 "s"(a.v_out), "s"(a.idx), "s"(a.all_idx), "s"(a.k), "s"(a.chunks));
    const uint32_t kv = blockIdx.y >= (uint32_t)a.n_kv_heads ? 1u : 0u, h = blockIdx.y - kv * (uint32_t)a.n_kv_heads;
    const uint32_t li = blockIdx.z;
    const uint32_t r = div_by(blockIdx.x, a.chunks, a.inv_chunks);
    char* const head_out =
        static_cast<char*>(kv ? a.v_out : a.k_out) + (uint64_t)(li * (uint32_t)a.n_kv_heads + h) * (uint64_t)a.head_out_bytes;
    if (r >= (uint32_t)a.k_eff) {  // uniform: one of the prefix blocks that end the x dimension
        const int64_t prefix_bytes = (int64_t)a.prefix_rows * a.head_dim * EB;
        copy_prefix((kv ? a.sys_v : a.sys_k) + ((int64_t)li * a.n_kv_heads + h) * prefix_bytes, head_out, prefix_bytes,
                    blockIdx.x - (uint32_t)a.k_eff * a.chunks);
        return;
    }
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;  // not written by this launch where it is read
    uint32_t t;
    if constexpr (SELECT > 0) {
        __shared__ uint32_t chosen;
        __shared__ SelectScratch<SELECT> shared;
        if (SELECT == kBlock / 64 || tid < 64 * SELECT) {
            const int lane = (int)(tid & 63u), wave = SELECT == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(tid >> 6));
            uint32_t key[kSelectKeys];
            load_keys_of_row<kSelectKeys>(a.scores + (int64_t)li * a.score_stride, a.n_groups, wave, lane, key);
            select_largest<SELECT, kSelectKeys>(key, a.k_eff, wave, lane, &shared, [&](uint32_t rank, int i) {
                if (rank == r) chosen = (uint32_t)i;  // one lane: ranks are distinct and r < k_eff
            });
        }
        __syncthreads();
        t = (uint32_t)__builtin_amdgcn_readfirstlane((int)chosen);
    } else {
        t = a.all_idx ? r : ((scalar_ptr)(uintptr_t)a.idx)[(uint64_t)li * (uint32_t)a.k + r];
    }
    if (t >= (uint32_t)a.n_groups) return;  // not a stored group: leave the rows alone

    const uint32_t begin = (blockIdx.x - r * a.chunks) * a.chunk_items;
    const uint32_t end = min(a.tile_items, begin + a.chunk_items);
    const uint64_t tile = (uint64_t)((a.layer0 + li) * 2u + kv) * a.plane_tiles + (uint64_t)t * (uint32_t)a.n_kv_heads + h;
    const char* const codes_t = reinterpret_cast<const char*>(a.codes) + tile * (a.tile_items * CW);
    const char* const meta_t = static_cast<const char*>(a.meta) + tile * a.tile_meta_bytes;
    char* const out = head_out + a.prefix_bytes + (uint64_t)r * (a.tile_items * (N * EB));
    const uint32_t first = begin + tid;
    const bool active = !TOKEN_AXIS || tid < a.step;
    f32x2 ch[N];  // token axis: the pairs of this lane's channels, loaded once
    if (TOKEN_AXIS) {
        const uint32_t slot = tid - div_by(tid, a.lanes_per_row, a.inv_lanes_per_row) * a.lanes_per_row;
#pragma unroll
        for (int i = 0; i < N; ++i) ch[i] = widen_pair(reinterpret_cast<const meta_pair*>(meta_t)[slot * N + i]);
    }

    uint32_t w[kUnroll];
    meta_pair sm[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const uint32_t item = first + u * a.step;
        w[u] = 0u;
        sm[u] = meta_pair{};
        if (active && item < end) {
            w[u] = load_codes<BITS, N, SELECT == kPastCaches>(codes_t + item * CW);
            if (!TOKEN_AXIS)
                sm[u] = *reinterpret_cast<const meta_pair*>(meta_t + (item >> a.lpg_shift) * (uint32_t)sizeof(meta_pair));
        }
    }
    // One wait for all loads.  Without it each item waits for its own, which after the first store is a wait for that store as well: 28 layers x 64
    // groups x 196 x 128 (by pieces now) 163.5 -> 162 us, 73 tokens x 13 groups 3 % less; but the token axis, with more items a lane, and float32
    // output are 2 to 5 % slower with it.
    if constexpr (!TOKEN_AXIS && EB == 2) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0) alone
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const uint32_t item = first + u * a.step;
        if (active && item < end) {
            float x[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float c = (float)((w[u] >> (BITS * i)) & CMASK);
                const f32x2 p = TOKEN_AXIS ? ch[i] : widen_pair(sm[u]);
                x[i] = __builtin_fmaf(c, p[0], p[1]);  // Eq. 11, rounded once to float32
            }
            store_items(out + item * (N * EB), OUT{}, x);
        }
    }
    if (SELECT > 0 && blockIdx.y == 0 && begin == 0 && tid == 0) a.sel_idx[(int64_t)li * a.k + r] = (int32_t)t;
    // last, so that the index load above stays a scalar load
    if (SELECT <= 0 && a.all_idx && blockIdx.y == 0 && begin == 0 && tid == 0) a.all_idx[(int64_t)li * a.k + r] = (int32_t)r;
}

// ------------------------------------------------------------------ the gather by pieces of its output
// Large launches of the head_dim axis, and those of the smallest tiles (gather_by_pieces in oqm_dispatch.h).  What bounds them is the order in which
// memory is written: plain 16-byte stores of 755 MB take 112 us where every workgroup writes the next 4 KB, 124 where it writes 16 KB, 153 with 64 KB
// and 180 from a persistent grid.  Tiles and their chunks are not multiples of 4 KB, so here the rows of a head are cut into aligned pieces of 4 KB
// whatever tile they belong to, and a workgroup takes kPieces of them, eight pieces apart: workgroups go round-robin over the eight XCDs, so that the
// ones in flight write one dense window of which each XCD has every eighth piece.  Two pieces hide the loads; with one a wave lives too short for
// them, three or four open the window. A wave's 64 items lie in at most two tiles.  Buffer instructions drop what lies outside of the rows, so
// nothing branches. 28 layers x 4 heads x 196 x 128 x 64 groups (944 MB), codes and pairs of random bits, one store, us: chunks 158, one piece 185,
// two 156.2, three 157, four 158.6; an arithmetic-free kernel of the same order with nothing but this shape's constants 153.4 (two adjacent pieces
// 157; runs of 16 workgroups per XCD 155; 512 threads 156, 1024 172; index loads per lane 174). 128 groups (quant-groups of 32, 2.0 GB) 337 -> 325;
// 37 x 256, 700 MB of output 162 -> 152; 61 x 96 168 -> 162. The last round of a head shares what is left of its pieces, first half and second half,
// among as few workgroups: with whole rounds alone a head of 785 pieces (64 groups behind a prefix) left seven of 400 workgroups idle, one of 304 16
// of 160.  Tiles / whole rounds / this, three stores in turn: 64 groups behind 14 rows 157.5 / 159.0 / 156.2, in buffers that start 512 bytes behind
// a piece 157.5 / 157.0 / 156.0, 72 176.4 / 180.9 / 174.5; 8 heads of 50 x 128, 97 groups 123.8 / 126.7 / 120.2, behind 14 rows 125.5 / 120.8 /
// 119.8.  Rounds that start on 32 KB of every head, so that an XCD keeps to the same eighth of memory over all heads: 159 at 64 groups behind 14
// rows, 177.7 at 72.
// What the kernel needs of a DequantArgs, made on the host.
struct PieceArgs {
    const char *codes, *meta;  // of the first layer asked for
    const int32_t* idx;        // or, where every stored group is taken in order, where these indices go
    char *k_out, *v_out;       // behind the prefix rows of the first head
    uint64_t code_plane, meta_plane, head_out_bytes;        // bytes of a (layer, K|V); of a head's active buffer
    uint32_t code_tile, meta_tile, code_group, meta_group;  // bytes of a tile, of the tiles of a group
    uint32_t tile_items, inv_tile_items, k_eff, n_groups;
    uint32_t k, heads, blocks, pair_shift;
    const char *sys_k, *sys_v;
    uint64_t prefix_bytes;
};

constexpr int kNonTemporal = 2;  // cache policy of the buffer builtins

template <int BYTES, bool PAST>
__device__ __forceinline__ uint32_t buffer_codes(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    constexpr int aux = PAST ? kNonTemporal : 0;
    if constexpr (BYTES == 4) return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, aux);
    else if constexpr (BYTES == 2) return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, aux);
    else return (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, (int)off, 0, aux);
}
__device__ __forceinline__ void buffer_pair(__amdgpu_buffer_rsrc_t r, uint32_t off, f32x2& p) {
    p = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
__device__ __forceinline__ void buffer_pair(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t& p) {
    p = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}
// Memory from `base` on, raw: byte offsets, and what lies past `bytes` is read as zero and not written.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const char* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)bytes, 0x00020000);
}

// grid (a workgroup for two pieces, then prefix blocks; K heads, then V heads; layer).  ALL: every stored group is taken in order, and
// these indices are written.
template <typename OUT, int N, int BITS, bool MB, bool PAST_CACHES, bool ALL>
__global__ void __launch_bounds__(kBlock) dequant_gather_pieces_kernel(const PieceArgs a) {
    constexpr uint32_t CW = BITS * N / 8;  // bytes of packed codes per item
    constexpr uint32_t CMASK = (1u << BITS) - 1u;
    constexpr uint32_t kItemBytes = 16;
    typedef typename MetaPair<MB>::type meta_pair;  // two float32, or two bfloat16 in one word
    // everything the addresses need is requested at once, not behind the index
    asm volatile("" ::"s"(a.codes), "s"(a.meta), "s"(a.idx), "s"(a.k_out), "s"(a.v_out), "s"(a.code_plane), "s"(a.meta_plane), "s"(a.head_out_bytes),
                 "s"(a.code_tile), "s"(a.meta_tile), "s"(a.code_group), "s"(a.meta_group), "s"(a.tile_items), "s"(a.inv_tile_items), "s"(a.k_eff), "s"(a.n_groups),
                 "s"(a.k), "s"(a.heads), "s"(a.blocks), "s"(a.pair_shift));
    const uint32_t kv = blockIdx.y >= a.heads ? 1u : 0u, h = blockIdx.y - kv * a.heads, li = blockIdx.z, head = li * a.heads + h;
    char* const out0 = kv ? a.v_out : a.k_out;
    if (blockIdx.x >= a.blocks) {  // uniform: one of the prefix blocks that end the x dimension
        copy_prefix((kv ? a.sys_v : a.sys_k) + head * a.prefix_bytes, out0 + head * a.head_out_bytes - a.prefix_bytes, (int64_t)a.prefix_bytes,
                    blockIdx.x - a.blocks);
        return;
    }
    const uint32_t lane = threadIdx.x & 63u, ti = a.tile_items, last = a.k_eff - 1u;
    // items between the start of the first piece and the rows
    const uint32_t lead = (((uint32_t)(uintptr_t)out0 + head * (uint32_t)a.head_out_bytes) & (kBlock * kItemBytes - 1u)) / kItemBytes;
    // items between a workgroup's pieces; the last round of a head has what is left of its workgroups
    const uint32_t round = blockIdx.x & ~(kXcds - 1u), apart = min(kXcds, a.blocks - round) * kBlock;
    // first item of the wave, of the first piece; below zero in front of the rows
    const uint32_t first = (round * kPieces + (blockIdx.x & (kXcds - 1u))) * kBlock +
                           ((uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~63u) - lead;
    if ((int)first >= (int)(a.k_eff * ti)) return;  // uniform in a wave: a last piece that only other heads have
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;  // not written by this launch where it is read
    typedef const __attribute__((address_space(4))) char* scalar_bytes;
    const scalar_bytes idx = (scalar_bytes)(uintptr_t)a.idx;
    uint32_t r[kPieces], t[kPieces][2];  // rank of the wave's first tile; groups of it and of the next
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
        r[p] = min(div_by((uint32_t)max((int)(first + p * apart), 0), ti, a.inv_tile_items), last);
        const uint32_t next = min(r[p] + 1u, last);
        t[p][0] = ALL ? r[p] : *(scalar_ptr)(idx + (li * a.k + r[p]) * 4u);
        t[p][1] = ALL ? next : *(scalar_ptr)(idx + (li * a.k + next) * 4u);
    }
    const uint32_t plane = li * 2u + kv;
    const __amdgpu_buffer_rsrc_t codes = buffer(a.codes + plane * a.code_plane + h * a.code_tile, (uint32_t)a.code_plane - h * a.code_tile);
    const __amdgpu_buffer_rsrc_t pairs = buffer(a.meta + plane * a.meta_plane + h * a.meta_tile, (uint32_t)a.meta_plane - h * a.meta_tile);
    const __amdgpu_buffer_rsrc_t rows = buffer(out0 + head * a.head_out_bytes, a.k_eff * ti * kItemBytes);
    uint32_t w[kPieces], to[kPieces];
    meta_pair sm[kPieces];
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
        const uint32_t item = first + p * apart + lane, at = item - r[p] * ti;
        const bool second = (int)at >= (int)ti;
        // offsets of the tile that item 0 of the wave's first tile would have
        const uint32_t c0 = t[p][0] * a.code_group, c1 = t[p][1] * a.code_group - a.code_tile;
        const uint32_t m0 = t[p][0] * a.meta_group, m1 = t[p][1] * a.meta_group - a.meta_tile;
        w[p] = buffer_codes<CW, PAST_CACHES>(codes, (second ? c1 : c0) + at * CW);
        buffer_pair(pairs, (second ? m1 : m0) + (at >> a.pair_shift) * (uint32_t)sizeof(meta_pair), sm[p]);
        // not a stored group: leave the rows alone
        to[p] = (second ? t[p][1] : t[p][0]) < a.n_groups ? item * kItemBytes : 0xffffffffu;
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0) alone: one wait for all loads, so that no store is waited for
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
        float x[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float c = (float)((w[p] >> (BITS * i)) & CMASK);
            const f32x2 pair = widen_pair(sm[p]);
            x[i] = __builtin_fmaf(c, pair[0], pair[1]);  // Eq. 11, rounded once to float32
        }
        __builtin_amdgcn_raw_buffer_store_b128(pack_items(OUT{}, x), rows, (int)to[p], 0, kNonTemporal);
    }
    if (ALL && blockIdx.y == 0) {
#pragma unroll
        for (int p = 0; p < kPieces; ++p) {
            const uint32_t item = first + p * apart + lane, at = item - r[p] * ti, rank = r[p] + (at == ti ? 1u : 0u);
            if ((int)item >= 0 && (at == 0u || at == ti) && rank <= last) const_cast<int32_t*>(a.idx)[(uint64_t)li * a.k + rank] = (int32_t)rank;
        }
    }
}

template <typename OUT, int N>
hipError_t launch_pieces(const DequantArgs& a, uint32_t prefix_blocks, hipStream_t s) {
    PieceArgs f{};
    f.code_tile = a.tile_items * (uint32_t)(N * a.bits / 8);
    f.meta_tile = a.tile_meta_bytes;
    f.code_plane = (uint64_t)a.plane_tiles * f.code_tile;
    f.meta_plane = (uint64_t)a.plane_tiles * f.meta_tile;
    f.code_group = f.code_tile * (uint32_t)a.n_kv_heads;
    f.meta_group = f.meta_tile * (uint32_t)a.n_kv_heads;
    f.codes = reinterpret_cast<const char*>(a.codes) + 2u * (uint64_t)a.layer0 * f.code_plane;
    f.meta = static_cast<const char*>(a.meta) + 2u * (uint64_t)a.layer0 * f.meta_plane;
    f.idx = a.all_idx ? a.all_idx : a.idx;
    f.k_out = static_cast<char*>(a.k_out) + a.prefix_bytes;
    f.v_out = static_cast<char*>(a.v_out) + a.prefix_bytes;
    f.head_out_bytes = (uint64_t)a.head_out_bytes;
    f.tile_items = a.tile_items;
    f.inv_tile_items = reciprocal_u32(a.tile_items);
    f.k_eff = (uint32_t)a.k_eff;
    f.n_groups = (uint32_t)a.n_groups;
    f.k = (uint32_t)a.k;
    f.heads = (uint32_t)a.n_kv_heads;
    f.pair_shift = a.lpg_shift;
    f.sys_k = a.sys_k;
    f.sys_v = a.sys_v;
    f.prefix_bytes = (uint64_t)a.prefix_bytes;
    f.blocks = (uint32_t)piece_blocks(a);
    const dim3 grid(f.blocks + prefix_blocks, 2 * f.heads, a.n_layers);
    auto go = [&](auto bits, auto mb, auto past) {
        constexpr int B = decltype(bits)::value;
        constexpr bool M = decltype(mb)::value, C = decltype(past)::value;
        if (a.all_idx) launch(dequant_gather_pieces_kernel<OUT, N, B, M, C, true>, grid, dim3(kBlock), 0, s, f);
        else launch(dequant_gather_pieces_kernel<OUT, N, B, M, C, false>, grid, dim3(kBlock), 0, s, f);
        return hipGetLastError();
    };
    using std::integral_constant;
    if constexpr (N == 8) {
        auto four = [&](auto mb) {
            return gather_past_caches(a) ? go(integral_constant<int, 4>{}, mb, std::true_type{}) : go(integral_constant<int, 4>{}, mb, std::false_type{});
        };
        if (a.bits == 4) return a.meta_bf16 ? four(std::true_type{}) : four(std::false_type{});
    }
    return a.meta_bf16 ? go(integral_constant<int, 2>{}, std::true_type{}, std::false_type{})
                       : go(integral_constant<int, 2>{}, std::false_type{}, std::false_type{});
}

// The prefix alone.  grid (chunks, H_k * n_layers, 2).
__global__ void __launch_bounds__(kBlock) prefix_copy_kernel(const DequantArgs a, const int64_t head_bytes,
                                                             const int64_t prefix_bytes) {
    copy_prefix((blockIdx.z ? a.sys_v : a.sys_k) + (int64_t)blockIdx.y * prefix_bytes,
                static_cast<char*>(blockIdx.z ? a.v_out : a.k_out) + (int64_t)blockIdx.y * head_bytes, prefix_bytes,
                blockIdx.x);
}

template <typename OUT>
hipError_t prefix_copy(const DequantArgs& a, hipStream_t s) {
    constexpr int64_t eb = elem_bytes<OUT>::value;
    const int64_t prefix_bytes = (int64_t)a.prefix_rows * a.head_dim * eb;  // multiple of 16: d % 8 == 0
    const int64_t head_bytes = ((int64_t)a.prefix_rows + (int64_t)a.k * a.group_tokens) * a.head_dim * eb;
    if (prefix_bytes == 0 || a.n_layers == 0) return hipSuccess;
    const int64_t chunks = (prefix_bytes / 16 + kBlock - 1) / kBlock;
    if (chunks > 0x7fffffffLL || (int64_t)a.n_kv_heads * a.n_layers > 65535) return hipErrorInvalidValue;
    launch(prefix_copy_kernel, dim3((unsigned)chunks, a.n_kv_heads * a.n_layers, 2), dim3(kBlock), 0, s, a, head_bytes,
                                                                                                     prefix_bytes);
    return hipGetLastError();
}

template <typename OUT, uint32_t N>
hipError_t launch_t(const DequantArgs& args, hipStream_t s) {
    if (args.n_layers == 0 || args.k_eff == 0) return hipSuccess;
    DequantArgs a = args;
    constexpr uint32_t eb = elem_bytes<OUT>::value;
    const bool tok = a.qaxis == TOM_QAXIS_TOKENS;
    const uint32_t lpr = (uint32_t)a.head_dim / N, G = (uint32_t)a.group_tokens;
    a.lanes_per_row = lpr;
    a.inv_lanes_per_row = reciprocal_u32(lpr);
    a.step = tok ? kBlock / lpr * lpr : kBlock;
    a.tile_items = G * lpr;  // G * d * 4 < 2^31 is checked by the API layer
    const uint32_t passes = (a.tile_items + a.step - 1) / a.step;
    // Up to `whole` passes one workgroup takes the tile, above that equal chunks (whole rows) of at most `most`.  On the token axis every lane first
    // loads the pairs of its channels, 64 bytes at 16-bit output against 16 stored per pass, so it takes more passes, but for launches that leave
    // most compute units without a tile.  28 layers, us per question (200 stored groups, 10 to 60 selected), chunks of at most 3 / 4 / 5 passes:
    // head_dim axis bf16 109.0 / 110.6 / 111.8, float32 105 / 101.7 / 112; token axis float32 88.7 / 97 / 100.  Token axis bf16, 64 of 200 groups,
    // chunks of at most 3 / 4 / 5 passes and the tile whole, three stores in turn: 80 x 128 (5 passes) 85 / 85 / 74, 100 x 128 (7) 109 / 93 / 93 /
    // 94, 112 x 128 (7) 113 / 101 / 101 / 105, 196 x 128 (13) 182 / 172 / 161; the same question again: 58 / 58 / 62, 72 / 68 / 68 / 77, 75 / 80 / 80
    // / 88, 163 / 143 / 148; 32 groups 35 / 35 / 34, 43 / 39 / 39 / 42, 45 / 44 / 44 / 46, 65 / 66 / 71.  One group of one layer, 8 tiles: 9.0 / 9.0
    // / 9.5, 9.0 / 9.3 / 9.3 / 9.9, 9.1 / 9.3 / 9.3 / 9.9, 9.0 / 9.3 / 9.5; 64 tiles 0.1 to 0.4 apart, 256 level. Six and seven passes in two
    // workgroups / whole, while a round of the chip (2048) holds the whole tiles: 96 x 128 (6 passes) 5 groups (1120 tiles) 15.4 / 13.9, 8 (1792)
    // 17.3 / 16.9, 10 (2240) 20.5 / 20.5, 16 26.0 / 25.4, 64 65 / 74; 150 x 80 10 20.6 / 22.0; 100 x 128 (7) 6 17.7 / 16.4, 8 19.2 / 18.5; of 700
    // groups 8 25.3 / 23.7, 10 27.3 / 28.1, 32 45 / 48.
    const int64_t tiles = (int64_t)a.n_layers * 2 * a.n_kv_heads * a.k_eff;
    const bool many = tok && eb == 2 && tiles > 128;
    // float32, token axis, chunks of at most 3 / 4, three stores in turn: 50 x 128 (7 passes) 600 MB 137 / 123, 250 45.1 / 43.9, 100 19.0 / 18.3 (the
    // same question again 16.7 / 17.1); 80 x 128 (10) 600 MB 123 / 108; 112 x 128 (14) 107 / 111, 196 x 128 105 / 114.
    const bool four = !tok || (passes <= 10 && tiles * a.tile_items * 16 >= 200000000);
    const uint32_t whole = many ? (tiles <= 2048 ? 7 : 5) : 4, most = eb == 2 ? (many ? 5 : 3) : (four ? 4 : 3);
    const uint32_t fit = passes <= whole ? whole : most;
    a.chunks = passes <= whole ? 1 : (passes + most - 1) / most;
    while ((G + a.chunks - 1) / a.chunks * lpr > fit * a.step) ++a.chunks;
    a.chunk_items = (G + a.chunks - 1) / a.chunks * lpr;
    const uint32_t unroll = (a.chunk_items + a.step - 1) / a.step;  // at most fit
    a.inv_chunks = reciprocal_u32(a.chunks);
    if (N < 8 && (int64_t)a.k_eff * a.chunks * kBlock >= 1LL << 31) return launch_t<OUT, 8>(args, s);  // fewer, longer workgroups
    if ((int64_t)a.k_eff * a.chunks > 0x7fffffffLL) return hipErrorInvalidValue;
    a.lpg_shift = 0;
    while (!tok && ((int)N << a.lpg_shift) < a.qgroup) ++a.lpg_shift;  // qgroup is a power of two
    a.tile_meta_bytes = (tok ? (uint32_t)a.head_dim : G * (lpr >> a.lpg_shift)) * (a.meta_bf16 ? 4u : 8u);
    a.plane_tiles = (int64_t)a.capacity_groups * a.n_kv_heads;
    a.prefix_bytes = (int64_t)a.prefix_rows * a.head_dim * eb;
    a.head_out_bytes = a.prefix_bytes + (int64_t)a.k * a.group_tokens * a.head_dim * eb;
    const int select = a.scores ? select_waves(a) : 0;
    if (a.scores && !select)
        if (hipError_t e = launch_topk(a.scores, a.score_stride, a.n_layers, a.n_groups, a.k, a.k_eff, TOM_ORDER_INDEX_ASC,
                                       a.sel_idx, s))
            return e;
    uint32_t prefix_blocks = 0;
    if (a.sys_k && a.prefix_rows > 0) {
        if (prefix_joins_gather(a)) {
            prefix_blocks = (uint32_t)((a.prefix_bytes / 16 + kBlock - 1) / kBlock);
        } else if (hipError_t e = prefix_copy<OUT>(a, s)) {
            return e;
        }
    }
    if constexpr (N * eb == 16) {
        if (!select && gather_by_pieces(a, eb == 2, prefix_blocks)) return launch_pieces<OUT, N>(a, prefix_blocks, s);
    }
    const dim3 grid((uint32_t)a.k_eff * a.chunks + prefix_blocks, 2 * a.n_kv_heads, a.n_layers), block(kBlock);
    auto go = [&](auto unroll, auto tokens, auto bits, auto mb) {
        constexpr int U = decltype(unroll)::value, B = decltype(bits)::value;
        constexpr bool K = decltype(tokens)::value, M = decltype(mb)::value;
        if constexpr (!K && B == 4 && eb == 2) {
            if (!select && gather_past_caches(a)) return launch(dequant_gather_kernel<OUT, N, U, K, B, M, kPastCaches>, grid, block, 0, s, a);
        }
        if (!select) launch(dequant_gather_kernel<OUT, N, U, K, B, M, 0>, grid, block, 0, s, a);
        else if (select == 1) launch(dequant_gather_kernel<OUT, N, U, K, B, M, 1>, grid, block, 0, s, a);
        else launch(dequant_gather_kernel<OUT, N, U, K, B, M, kBlock / 64>, grid, block, 0, s, a);
    };
    auto with_storage = [&](auto unroll, auto tokens) {
        if (a.bits == 2 && a.meta_bf16) go(unroll, tokens, std::integral_constant<int, 2>{}, std::true_type{});
        else if (a.bits == 2) go(unroll, tokens, std::integral_constant<int, 2>{}, std::false_type{});
        else if (a.meta_bf16) go(unroll, tokens, std::integral_constant<int, 4>{}, std::true_type{});
        else go(unroll, tokens, std::integral_constant<int, 4>{}, std::false_type{});
    };
    if (!tok) {
        if (unroll <= 3) with_storage(std::integral_constant<int, 3>{}, std::false_type{});
        else with_storage(std::integral_constant<int, 4>{}, std::false_type{});
    } else {
        if (unroll <= 3) with_storage(std::integral_constant<int, 3>{}, std::true_type{});
        else if (unroll == 4) with_storage(std::integral_constant<int, 4>{}, std::true_type{});
        else if constexpr (eb == 2) {
            if (unroll == 5) with_storage(std::integral_constant<int, 5>{}, std::true_type{});
            else with_storage(std::integral_constant<int, 7>{}, std::true_type{});
        }
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_prefix_copy(const DequantArgs& args, const void* sys_k, const void* sys_v, int out_dtype,
                              hipStream_t s) {
    DequantArgs a = args;
    a.sys_k = static_cast<const char*>(sys_k);
    a.sys_v = static_cast<const char*>(sys_v);
    return out_dtype == TOM_F32 ? prefix_copy<In_f32>(a, s) : prefix_copy<In_bf16>(a, s);
}

hipError_t launch_dequant_gather(const DequantArgs& a, int out_dtype, hipStream_t s) {
    if (a.k_eff == 0) return hipSuccess;
    switch (out_dtype) {
        // a lane keeps its channels on the token axis, and a row has to fit the workgroup
        case TOM_F32: return a.head_dim / 4 <= kBlock ? launch_t<In_f32, 4>(a, s) : launch_t<In_f32, 8>(a, s);
        case TOM_BF16: return launch_t<In_bf16, 8>(a, s);
        case TOM_F16: return launch_t<In_f16, 8>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace oqm
