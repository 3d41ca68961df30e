// vpp_chunk_attn.hip -- chunked-prefill causal attention for MI355X (gfx950).
//
// Computes Eq. (1) of the paper (section 2.1), softmax(Q K^T * scale) V under
// the causal rule, for one chunk of query tokens at in-request positions
// prefix .. prefix+len-1 attending to the cached prefix plus the chunk itself
// (section 2.4). Several requests may share a chunk (packing, section 5.3).
//
// Kernel layout: one workgroup = 4 waves running one work slot of one group of
// query heads that share a kv head: one query tile of 256 (or 128) rows -- a row
// is a token of one of those heads -- of one segment, or two, the first with its
// keys ascending, the second -- its partner from the other end of the segment --
// descending, so that the workgroups on an XCD read the same keys at the same
// time. Keys stream through LDS 64 at a time:
//   * S^T = K Q^T on v_mfma_f32_32x32x16_bf16: keys are the M dimension,
//     queries the N dimension, head dim the K dimension. Each lane then owns
//     one query (column lane%32) and 16 keys per 32-key block, so a row max or
//     row sum needs only one exchange with lane^32.
//   * Online softmax in fp32 with exp2 (scale folded with log2 e).
//   * O^T = V^T P^T on the same MFMA: P leaves the S^T accumulators already in
//     the B-operand layout (no shuffles); each lane reads its 8 keys of one
//     value column from the row-major V tile with two transposing 8-byte LDS
//     reads (ds_read_b64_tr_b16).
//   * Only key tiles that cross the diagonal (or the end of the key range) are
//     masked; every wave computes every key tile of its workgroup's range.
//   * Split-KV: the prefix of a segment may be cut into pieces whose fp32
//     partial results are merged by their log-sum-exp in a second pass.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <type_traits>
#include <mutex>
#include <new>
#include <vector>

#include "vpp_chunk_attn.h"

// VPP_PART: 0 = host code and the contiguous-cache kernels, 1 = the paged-cache
// kernels, 2 = the split-key-layout kernels, 4 = the host code alone (for a test that
// replays launches on the CPU); unset (3) = everything in one translation unit.
#ifndef VPP_PART
#define VPP_PART 3
#endif

namespace {

constexpr int BN = 64;         // keys per inner step
constexpr int NWAVES = 4;
// query rows per workgroup tile: 4 waves x NB blocks of 32 rows
constexpr int block_rows(int nb) { return 32 * nb * NWAVES; }
[[maybe_unused]] constexpr int BM_MAX = block_rows(2);
constexpr int NTHREADS = 64 * NWAVES;
[[maybe_unused]] constexpr int MAX_SPLITS = 16;  // a fixed split request
[[maybe_unused]] constexpr int STAGING_SLOTS = 4;
// cache layouts (kernel template argument KVM)
[[maybe_unused]] constexpr int KV_CONTIG = 0, KV_PAGED = 1, KV_ROPE = 2;
// split key layout: granules of the per-head and of the shared part of a K row
constexpr int NOPE_GR = 16, ROPE_GR = 8;
// Lazy rescale: the running max used for exp2 is refreshed only when a row's
// max grows past it by more than this many powers of two; O and l share the
// stale max, so the final quotient is unchanged and P stays <= 2^TAU.
constexpr float LAZY_TAU = 8.0f;
// The next tiles' global->LDS copies are spread over the first 1/LOAD_SPREAD
// of a tile's MFMA slots.
constexpr int LOAD_SPREAD = 2;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// Word 3 of a raw buffer resource (untyped 32-bit data, no swizzle).
constexpr int BUFFER_RSRC_WORD3 = 0x00020000;
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// Raw buffer resource over [base, base + bytes): reads past the end return 0.
__device__ __forceinline__ i32x4 make_rsrc(const void* base, int32_t bytes) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)b);
    r[1] = __builtin_amdgcn_readfirstlane((int32_t)((uint32_t)(b >> 32) & 0xffffu));  // stride 0
    r[2] = __builtin_amdgcn_readfirstlane(bytes);
    r[3] = BUFFER_RSRC_WORD3;
    return r;
}

// 16 bytes per lane from global memory (resource + per-lane byte offset)
// straight into LDS at lds_addr + 16*lane. Written as inline asm on purpose:
// the compiler then does not track these copies as pending LDS writes and
// inserts no wait for them in front of later LDS reads of other buffers; the
// kernel waits for them itself (vmcnt) before the barrier that publishes the
// buffer they fill. Nothing else in the kernel keeps a value in M0.
// NT: non-temporal, for tiles that no other workgroup reads (see Launch::nt).
template <int OFF, bool NT>
__device__ __forceinline__ void copy16_to_lds(const i32x4& rsrc, uint32_t lds_base, uint32_t voff) {
    // M0 = lds_base + OFF: one live SGPR for every copy of the kernel.
    // The scalar add also writes SCC: without the clobber the compiler may
    // place a copy between the two halves of a 64-bit scalar add and the high
    // half then adds the copy's carry instead of its own (an address 4 GiB off
    // whenever the low half wraps).
    if constexpr (NT)
        asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                     :
                     : "s"(lds_base), "v"(voff), "s"(rsrc), "i"(OFF)
                     : "memory", "scc");
    else
        asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(lds_base), "v"(voff), "s"(rsrc), "i"(OFF)
                     : "memory", "scc");
}

typedef vpp_chunk_attn_work_item_t WorkItem;
static_assert(sizeof(WorkItem) == 32, "work item layout");

}  // namespace

namespace {
// First key of piece b of a p-key prefix cut into n tile-aligned pieces; the last
// piece runs on to each tile's own end (its keys within the chunk).
__host__ __device__ inline int32_t piece_begin(int32_t p, int n, int b) {
    return (int32_t)((uint32_t)(p / BN) * (uint32_t)b / (uint32_t)n * (uint32_t)BN);
}
}  // namespace

// Kernel argument blocks, shared by the translation units that instantiate
// the kernels (the build compiles this file once per part, in parallel).
namespace vpp_detail {

// One launch group: the workgroups of one segment, all heads, split pieces and
// work slots. Groups are contiguous runs of the grid, longest slots first.
struct LaunchGroup {
    int32_t wg0;        // the group's first workgroup
    int32_t row0;       // first chunk row of the segment
    int32_t len;        // rows of the segment
    int32_t prefix;     // in-request position of the first row
    int32_t kv_start;   // cache row of the request's position 0
    int32_t seg;        // block-table row (paged cache)
    int32_t pieces;     // split pieces of the prefix (piece_begin); negative: last_pieces_first
    int32_t part0;      // first row of piece 0's fp32 partials; < 0: final results
    int32_t slots;      // work slots per head group and piece: two tiles, or one when slots == tiles
    int32_t tiles;      // query tiles per head group
};
// A chunk of up to INLINE_GROUPS segments carries its table in the kernel
// arguments: the 2.5 KB travel with the dispatch packet, where an upload of its own
// costs a copy of 2 us and the gaps around it, 12 to 15 us a run. Kernel arguments
// end at 4 KB.
constexpr int INLINE_GROUPS = 64;
struct GroupTable {
    LaunchGroup g[INLINE_GROUPS];
};

struct AttnArgs {
    const LaunchGroup* groups;  // table in device memory; null: the second kernel argument
    int32_t num_groups;
    int32_t num_heads;
    const u16* q;
    const u16* k;
    const u16* v;
    u16* out;         // bf16, row*o_st + h*o_sh
    float* lse;       // fp32, h*lse_sh + row (nullable)
    float* part_o;    // fp32 partials of split segments [partial row][Hq][DV]
    float* part_lse;  // [partial row][Hq]
    // element strides (the host checks that they fit in 31 bits)
    int32_t q_st, q_sh, k_st, k_sh, v_st, v_sh, o_st, o_sh, lse_sh;
    int32_t group;     // Hq / Hkv
    // Query heads per tile. A tile's row r is token r / pack of the tile, head
    // r % pack of `pack` heads that read the same kv head; r / pack is
    // (r * pack_magic) >> 16.
    int32_t pack, pack_magic;
    int32_t tile_tokens;  // tokens per tile
    int32_t head_groups;  // Hq / pack
    float scale_log2;  // softmax scale * log2(e)
    int32_t xcd_remap;
    // Paged cache (PAGED kernels only). Cache row j of segment s is row
    // j & (2^page_shift - 1) of page block_table[s * bt_st + (j >> page_shift)];
    // kv_start is a multiple of the key tile, so no tile straddles a page (pages
    // hold >= 64 rows).
    const int32_t* block_table;
    int64_t bt_st;
    int64_t k_sp, v_sp;  // element strides between pages
    int32_t page_shift;
    int32_t num_pages;   // page indices are clamped below it
    // Split key layout (KV_ROPE kernels only): k holds the per-head 128 dims of
    // each key, k_rope [rows][64] the 64 dims shared by all heads.
    const u16* k_rope;
    int32_t kr_st;
};

// The merge of split partials: one entry per split segment, covering the
// workgroups from block0 on. Piece b of the segment's row r is partial row
// part0 + b*len + r.
struct CombineSeg {
    int32_t block0, row0, len, pieces, part0;
};
struct CombineTable {
    CombineSeg s[INLINE_GROUPS];
};
struct CombineArgs {
    const CombineSeg* segs;  // table in device memory; null: the second kernel argument
    const float* part_o;
    const float* part_lse;
    u16* out;
    float* lse;
    int64_t o_st, o_sh, lse_sh;
    int32_t num_segs, num_heads, blocks;
};

// A planned launch: both kernels' arguments and grids (merge.blocks = 0: no merge).
struct Launch {
    AttnArgs a;
    GroupTable groups;
    CombineArgs merge;
    CombineTable segs;
    int32_t nb, dqk;
    // Whether most of the launch's key steps are of segments with one tile a kv head,
    // whose K/V tiles no other workgroup reads: their copies are then non-temporal
    // (128-row tiles only, which such launches use). Single tokens behind 4K to 23K
    // cached ones: 64 of 32/8 heads 635 -> 578 us, 16 of 16 MLA heads 194 -> 176; a
    // serving step with a 480-row prompt piece 257 -> 233. Where tiles share their keys
    // it costs time, the L2 keeping them too briefly: the tiles of a segment 1.5 to 6 %
    // (six short prompts 233 -> 247), the head groups of a kv head whose heads do not fit
    // one tile 5 to 19 % (32 single tokens of 32/1 heads 64 -> 75, of 71/1 791 -> 894).
    // With keys that come from memory, as in an engine, which reads the other layers' between
    // two calls on one: over 287 launches of single tokens non-temporal copies took 0.87 to
    // 1.1 times the time of others, mean 0.97. Keys still cached from the call before are
    // read up to 1.28 times slower.
    bool nt;
    int64_t workgroups;
};

hipError_t launch_attn_contig(const Launch& l, hipStream_t stream);
hipError_t launch_attn_paged(const Launch& l, hipStream_t stream);
hipError_t launch_attn_rope(const Launch& l, hipStream_t stream);

}  // namespace vpp_detail

namespace {

using vpp_detail::AttnArgs;
using vpp_detail::CombineArgs;
using vpp_detail::CombineSeg;
using vpp_detail::CombineTable;
using vpp_detail::GroupTable;
using vpp_detail::Launch;
using vpp_detail::LaunchGroup;
using vpp_detail::INLINE_GROUPS;

// LDS tiles: K [BN][DQK] and V [BN][DV] bf16, row-major in 16-byte granules,
// the granule index XOR-swizzled per row. The LDS serves 64 banks (256 bytes)
// per cycle:
//  * K is read by ds_read_b128, 16 lanes per cycle = 16 consecutive rows at one
//    logical granule; the 16 granules must fall on 16 different 16-byte bank
//    groups. With a multiple of 16 granules per row every row starts on the
//    same bank, so XOR with row & 15; with 8 (mod 16) granules per row
//    consecutive rows already alternate between the two 128-byte halves, so XOR
//    with (row >> 1) & 7 within each half.
//  * V is read by ds_read_b64_tr_b16, 32 lanes per cycle = 4 consecutive keys x
//    64 bytes; the four segments must fall in four different 64-byte quarters:
//    XOR with (key & 3) << 2 (16 granules per row), or with ((key >> 1) & 1) << 2
//    (8 granules per row, where odd keys already sit in the other half).
template <int KGR>
__device__ __forceinline__ int kswz(int row, int granule) {
    if constexpr (KGR % 16 == 0) return granule ^ (row & 15);
    else return granule ^ ((row >> 1) & 7);
}
template <int VGR>
__device__ __forceinline__ int vswz_bits(int key) {
    if constexpr (VGR % 16 == 0) return (key & 3) << 2;
    else return ((key >> 1) & 1) << 2;
}
template <int VGR>
__device__ __forceinline__ int vswz(int key, int granule) { return granule ^ vswz_bits<VGR>(key); }

// max of three floats in one v_max3_f32. Written as asm because the
// compiler's maxnum would first canonicalise every operand coming from an asm
// MFMA (one more VALU op per score); the scores are never NaN.
__device__ __forceinline__ float max3f(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Plain v_max_f32: the scores are never NaN (masked ones are -inf), so the
// canonicalising maxes fmaxf would add are not needed.
__device__ __forceinline__ float max2f(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float lane_swap32_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max2f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float lane_swap32_add(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS-only workgroup barrier: orders LDS traffic without waiting for the
// asynchronous global->LDS copies of the next stage.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// s_waitcnt with only vmcnt constrained (expcnt / lgkmcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Tables that travel in the kernel arguments or in device memory, read as
// constant memory: uniform indices become scalar loads.
typedef __attribute__((address_space(4))) const AttnArgs const_args_t;
typedef __attribute__((address_space(4))) const LaunchGroup const_group_t;
typedef __attribute__((address_space(4))) const CombineSeg const_seg_t;
template <typename T>
__device__ __forceinline__ T* const_ptr(uint64_t p) {
    return (T*)(uintptr_t)p;
}

// What a workgroup works on -- its table entry, tiles, keys and where the results go --
// is worked out by the functions from here to merge_place, on the host as well: a CPU
// test replays every workgroup of a launch through them.

// Search for the last of n table entries (their first word ascending, the first
// entry's <= x) whose first word is <= x: entries [lo, lo + cnt) are left. Each step
// compares 64 of them at once, one per lane: one step up to 64 entries, two up to 4096.
struct EntrySearch {
    int lo, cnt;
    __host__ __device__ int step() const { return (cnt + 63) >> 6; }
    __host__ __device__ bool has(int lane) const { return lane * step() < cnt; }
    __host__ __device__ int entry(int lane) const { return lo + min(lane * step(), cnt - 1); }  // a lane's entry
    __host__ __device__ void take(int hits) {  // how many lanes have an entry that is <= x
        const int s = step(), skip = (hits - 1) * s;
        lo += skip;
        cnt = min(s, cnt - skip);
    }
};
// The entry of x in a table of entries `stride` bytes apart.
__device__ __forceinline__ int find_entry(uint64_t table, int stride, int n, int x) {
    const int lane = threadIdx.x & 63;
    EntrySearch e{0, n};
    while (e.cnt > 1) {
        const int first =
            *(__attribute__((address_space(1))) const int32_t*)(uintptr_t)(table + (uint64_t)e.entry(lane) * stride);
        e.take(__popcll(__builtin_amdgcn_ballot_w64(e.has(lane) && first <= x)));
    }
    return __builtin_amdgcn_readfirstlane(e.lo);
}

// Workgroup i of a run of slots -> (slot, head); `heads` counts pieces too (the pieces of
// a head follow each other). Consecutive workgroups land on the 8 XCDs round robin.
// Where the slots are alike (two tiles each, or pieces without the tiles' own keys), each
// XCD gets a contiguous run of the head-major order, the slots of the same heads, which
// read the same K/V through that XCD's L2. Slots of one tile grow with their index: the
// XCDs that share a head take turns at its slots, longest first (contiguous runs gave one
// XCD the short half and the next the long half of a causal segment: 1120 us where turns
// take 921 and pairs 984, at 6915 rows and 64/4 heads). Every run is spread over all XCDs.
__host__ __device__ __forceinline__ void work_coords(int i, int slots, int heads, bool alike, bool remap, int& slot, int& head) {
    if (remap && alike) {
        const int n = slots * heads;
        const int x = i & 7;
        i = x * (n >> 3) + min(x, n & 7) + (i >> 3);
    } else if (remap) {
        const int g = min(3, __builtin_ctz(heads));  // XCDs x and x + 2^g share heads
        i = (i & ((1 << g) - 1)) * (heads >> g) * slots + (i >> g);
    }
    head = slots == 1 ? i : i / slots;
    slot = i - head * slots;
    if (!alike) slot = slots - 1 - slot;
}

// Token of a tile's row r, r < 256 (AttnArgs::pack_magic).
__host__ __device__ __forceinline__ int row_token(int r, int magic) { return (int)((uint32_t)r * (uint32_t)magic >> 16); }

// A workgroup's first (sub = 0) or second tile.
struct TileWork {
    int h, hk;                    // first query head, kv head
    int row0, nrows, pos0;        // first chunk row, rows (tokens), in-request position of the first
    int key_begin, key_end;       // keys of the request that this piece covers
    int out_row0;                 // where the results go: row0, or ~ the first partial row
};
struct TileArgs {  // of AttnArgs
    int32_t group, pack, tile_tokens, head_groups, xcd_remap;
};
// false: the workgroup has no such tile. `block` counts from the group's first workgroup.
__host__ __device__ __forceinline__ bool tile_work(const TileArgs& a, const LaunchGroup& g, int block, int sub, TileWork& w) {
    const int slots = g.slots, seg_tiles = g.tiles, pieces = abs(g.pieces);
    const bool paired = slots != seg_tiles;
    // the run's pieces: `per` of them, from `top` down (the last piece is the longest: first)
    int top = pieces - 1, per = pieces;
    bool alike = paired;
    if (g.pieces < 0) {  // two runs: the last pieces of all head groups, then the others
        const int last = slots * a.head_groups;
        if (block < last) {
            per = 1;
        } else {
            block -= last;
            --top, --per;
            alike = true;
        }
    }
    int slot, hg, piece = 0, piece_kb = 0, piece_ke = INT32_MAX;  // hg: head group
    work_coords(block, slots, a.head_groups * per, alike, a.xcd_remap != 0, slot, hg);
    if (pieces > 1) {
        const int hp = hg;
        hg = hp / per;
        piece = top - (hp - hg * per);
        piece_kb = piece_begin(g.prefix, pieces, piece);
        if (piece + 1 < pieces) piece_ke = piece_begin(g.prefix, pieces, piece + 1);
    }
    const int ti = sub == 0 ? slot : seg_tiles - 1 - slot;
    if (sub == 1 && (!paired || ti == slot)) return false;
    const int t_row0 = ti * a.tile_tokens;  // the tile's first token in the segment
    w.h = hg * a.pack;
    w.hk = a.pack == a.group ? hg : w.h / a.group;
    w.row0 = g.row0 + t_row0;
    w.nrows = min(a.tile_tokens, g.len - t_row0);
    w.pos0 = g.prefix + t_row0;
    w.key_begin = piece_kb;
    w.key_end = min(piece_ke, w.pos0 + w.nrows);
    w.out_row0 = g.part0 < 0 ? w.row0 : ~(g.part0 + piece * g.len + t_row0);
    return true;
}

template <int DQK, int DV, int NB>
struct Tiles {
    static constexpr int KS = DQK / 16;          // MFMA k-steps of S^T = K Q^T
    static constexpr int DB = DV / 32;           // 32-row blocks of O^T
    static constexpr int KGR = DQK / 8;          // 16-byte granules per K row
    static constexpr int VGR = DV / 8;
    static constexpr int K_BYTES = BN * KGR * 16;
    static constexpr int V_BYTES = BN * VGR * 16;
    static constexpr int BYTES = 2 * K_BYTES + 2 * V_BYTES;  // double-buffered K and V
    static constexpr int K_LOADS = BN * KGR / 64 / NWAVES;   // 16-byte loads per lane per tile
    static constexpr int V_LOADS = BN * VGR / 64 / NWAVES;
    static constexpr int NQK = 2 * KS * NB;      // MFMAs of one S^T tile (2 key blocks x NB query blocks)
    static constexpr int NPV = 4 * DB * NB;      // MFMAs of one O^T update (4 key groups x NB query blocks)
    static_assert(KGR % 8 == 0 && VGR % 8 == 0, "swizzle needs 8 granules per row");
    static_assert(BN * KGR % (64 * NWAVES) == 0 && BN * VGR % (64 * NWAVES) == 0, "whole wave loads");
};

// S^T MFMA i of a tile: key block mb = 1 first, so that the block-0
// accumulators of the next tile are written only after the softmax has
// consumed this tile's block 0 and their registers can be reused. Within a
// key block the k-steps run in order, each K fragment feeding NB MFMAs.
template <int KS, int NB>
struct QkCoords {
    static constexpr int mb(int i) { return 1 - i / (KS * NB); }
    static constexpr int ks(int i) { return (i % (KS * NB)) / NB; }
    static constexpr int nb(int i) { return i % NB; }
};

// ---------------------------------------------------------------------------
// Static instruction schedule of one key tile.
//
// One wave (one SIMD) runs, per tile, NQK MFMAs of the next tile's S^T, NPV
// MFMAs of this tile's O^T update and the softmax of this tile in fp32 VALU
// code. A wave issues in order; VALU work issued right after an MFMA runs
// while the matrix core is busy, so the softmax is cut into small atoms
// spread over the MFMA slots. With NB query blocks of 32 rows per wave:
//   atoms 0 .. 4NB-1      4 v_max3 steps of the row max per query block
//                         (block nb = a / 4)
//   atoms 4NB .. 5NB-1    finish the row max of block nb: lane exchange, lazy
//                         rescale decision, new reference max
//   atoms 5NB .. 37NB-1   one score each: exp2, row sum, bf16 packing;
//                         element e belongs to unit u = e / 8, which holds the
//                         8 P values one O^T MFMA consumes: query block
//                         nb = u % NB, 16-key group hh = (u / NB) % 2, key
//                         block mb = u / (2 NB)
// O^T MFMA p works on key group g = p / (NB*DB) (units g*NB .. g*NB+NB-1),
// value block d = (p / NB) % DB and query block nb = p % NB, so each V^T
// fragment feeds NB MFMAs in a row; it is placed only after its group's atoms.
// All atoms finish before the last group's MFMAs start.
// ---------------------------------------------------------------------------
template <int NB>
struct Atoms {
    static constexpr int N = 37 * NB;
    static constexpr int MAXF = 4 * NB;  // first finishing atom
    static constexpr int EXP = 5 * NB;   // first exp atom
    static constexpr int weight(int k) { return k < MAXF ? 24 : (k < EXP ? 70 : 23); }  // VALU cycles
    static constexpr int unit_last(int u) { return EXP + 8 * u + 7; }
};

template <int NQK, int NPV, int DB, int NB>
struct Schedule {
    typedef Atoms<NB> A;
    // the last tile has no next S^T to overlap with: it opens with one
    // VALU-only slot for the row max, then hides each key group's atoms under
    // the previous group's MFMAs
    static constexpr int NS = NQK + NPV + (NQK == 0 ? 1 : 0);
    static constexpr int GROUP_PV = NB * DB;  // O^T MFMAs per key group
    int kind[NS] = {};      // 0: S^T MFMA, 1: O^T MFMA, 2: no MFMA
    int index[NS] = {};     // S^T: see QkCoords; O^T: see above
    int atoms_end[NS] = {}; // atoms issued after slot s: [atoms_end[s-1], atoms_end[s])
    int rescale_before = 0; // slot before which the (rare) O rescale check runs
    constexpr Schedule() {
        int done_at[A::N] = {};
        if constexpr (NQK == 0) {
            kind[0] = 2;
            for (int k = 0; k < A::EXP + 8 * NB; ++k) done_at[k] = 0;
            for (int p = 0; p < NPV; ++p) {
                kind[1 + p] = 1;
                index[1 + p] = p;
            }
            for (int g = 1; g < 4; ++g)  // key group g under group g-1's MFMAs
                for (int j = 0; j < 8 * NB; ++j)
                    done_at[A::EXP + 8 * NB * g + j] = 1 + (g - 1) * GROUP_PV + (j * GROUP_PV) / (8 * NB);
        } else {
            // slot by which each atom is done: spread by weight over the slots
            // before the last group's MFMAs
            int total = 0;
            for (int k = 0; k < A::N; ++k) total += A::weight(k);
            const int span = NS - GROUP_PV;
            int acc = 0;
            for (int k = 0; k < A::N; ++k) {
                acc += A::weight(k);
                int s = (acc * span + total - 1) / total - 1;
                done_at[k] = s < 0 ? 0 : s;
            }
            // MFMA order: an O^T MFMA as soon as its key group's atoms are done, else an S^T MFMA
            int q = 0, p = 0;
            for (int s = 0; s < NS; ++s) {
                const int grp = p / GROUP_PV;
                const bool pv_ready = p < NPV && done_at[A::EXP - 1] < s &&
                                      done_at[A::unit_last(grp * NB + NB - 1)] < s;
                if (pv_ready || q >= NQK) {
                    kind[s] = 1;
                    index[s] = p++;
                } else {
                    kind[s] = 0;
                    index[s] = q++;
                }
            }
        }
        for (int s = 0; s < NS; ++s) {
            int n = 0;
            for (int k = 0; k < A::N; ++k) n += done_at[k] <= s;
            atoms_end[s] = n;
        }
        // The (rare) O rescale is a branch; it runs right after the finishing
        // atoms. Atoms scheduled between it and the first O^T MFMA feed only code
        // after the branch, and the compiler would sink them past it into one
        // burst with no MFMA to hide under.
        rescale_before = NS;
        for (int s = NS - 1; s >= 1; --s)
            if (atoms_end[s - 1] >= A::EXP) rescale_before = s;
        for (int s = NS - 1; s >= 0; --s)
            if (kind[s] == 1 && s < rescale_before) rescale_before = s;
    }
    // MFMA slots after the last S^T MFMA of the step
    constexpr int qk_tail() const {
        int last = -1;
        for (int s = 0; s < NS; ++s)
            if (kind[s] == 0) last = s;
        return NS - 1 - last;
    }
    // every O^T MFMA comes after the atoms it depends on; atoms run in order
    constexpr bool valid() const {
        for (int s = 0; s < NS; ++s) {
            if (s > 0 && atoms_end[s] < atoms_end[s - 1]) return false;
            if (kind[s] != 1) continue;
            const int grp = index[s] / GROUP_PV;
            const int before = s == 0 ? 0 : atoms_end[s - 1];
            if (before < A::unit_last(grp * NB + NB - 1) + 1) return false;
        }
        return atoms_end[NS - 1] == A::N;
    }
};

// The S^T MFMAs are inline asm so that each operand stays in the register
// file it belongs to for the whole loop: S in VGPRs (the softmax reads and
// writes it in place) and Q in AGPRs (only MFMAs read it). The compiler cannot
// see the latency of these instructions, so the schedule keeps the distance
// itself: an S^T tile is read by VALU code only in the next tile's step (after
// a barrier), and every step ends with at least four O^T MFMAs after its last
// S^T MFMA (checked in the kernel), each occupying the matrix core for longer
// than an S^T result takes to reach its registers. The O^T MFMAs use the
// builtin, so the compiler tracks their operand hazards (P packed by VALU code
// just before) and keeps O in AGPRs; the asm that rescales O in place runs only
// after an explicit drain.
#define MFMA_32x32x16_INIT(acc, a, b) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "a"(b))
#define MFMA_32x32x16_ACC(acc, a, b) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b))

__device__ __forceinline__ void mfma_drain() {
    // longer than the longest MFMA result latency: 3 x 16 wait states
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
}

// Load the KS B-operand fragments of a lane's NB query rows (16 bytes each, 32
// bytes apart) straight into AGPRs, where only MFMAs read them. Loading through
// VGPRs would leave a VGPR copy of Q alive across the whole loop. The wait stands in
// the same statement: the compiler takes the registers as written when it ends. It
// also covers the tile's first K and V copies, issued just before.
template <int KS, int NB>
__device__ __forceinline__ void load_q_agpr(bf16x8 (&qf)[NB][KS], const u16* const (&p)[NB]) {
    static_assert(KS == 4 || KS == 8 || KS == 12, "head dims 64, 128, 192");
    static_assert(NB == 1 || NB == 2, "query rows of a lane");
    if constexpr (KS == 4 && NB == 1) {
        asm volatile(
            "global_load_dwordx4 %0, %4, off\n\t"
            "global_load_dwordx4 %1, %4, off offset:32\n\t"
            "global_load_dwordx4 %2, %4, off offset:64\n\t"
            "global_load_dwordx4 %3, %4, off offset:96\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3])
            : "v"(p[0]) : "memory");
    } else if constexpr (KS == 4 && NB == 2) {
        asm volatile(
            "global_load_dwordx4 %0, %8, off\n\t"
            "global_load_dwordx4 %1, %8, off offset:32\n\t"
            "global_load_dwordx4 %2, %8, off offset:64\n\t"
            "global_load_dwordx4 %3, %8, off offset:96\n\t"
            "global_load_dwordx4 %4, %9, off\n\t"
            "global_load_dwordx4 %5, %9, off offset:32\n\t"
            "global_load_dwordx4 %6, %9, off offset:64\n\t"
            "global_load_dwordx4 %7, %9, off offset:96\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3]), "=a"(qf[1][0]),
              "=a"(qf[1][1]), "=a"(qf[1][2]), "=a"(qf[1][3])
            : "v"(p[0]), "v"(p[1]) : "memory");
    } else if constexpr (KS == 8 && NB == 1) {
        asm volatile(
            "global_load_dwordx4 %0, %8, off\n\t"
            "global_load_dwordx4 %1, %8, off offset:32\n\t"
            "global_load_dwordx4 %2, %8, off offset:64\n\t"
            "global_load_dwordx4 %3, %8, off offset:96\n\t"
            "global_load_dwordx4 %4, %8, off offset:128\n\t"
            "global_load_dwordx4 %5, %8, off offset:160\n\t"
            "global_load_dwordx4 %6, %8, off offset:192\n\t"
            "global_load_dwordx4 %7, %8, off offset:224\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3]), "=a"(qf[0][4]),
              "=a"(qf[0][5]), "=a"(qf[0][6]), "=a"(qf[0][7])
            : "v"(p[0]) : "memory");
    } else if constexpr (KS == 8 && NB == 2) {
        asm volatile(
            "global_load_dwordx4 %0, %16, off\n\t"
            "global_load_dwordx4 %1, %16, off offset:32\n\t"
            "global_load_dwordx4 %2, %16, off offset:64\n\t"
            "global_load_dwordx4 %3, %16, off offset:96\n\t"
            "global_load_dwordx4 %4, %16, off offset:128\n\t"
            "global_load_dwordx4 %5, %16, off offset:160\n\t"
            "global_load_dwordx4 %6, %16, off offset:192\n\t"
            "global_load_dwordx4 %7, %16, off offset:224\n\t"
            "global_load_dwordx4 %8, %17, off\n\t"
            "global_load_dwordx4 %9, %17, off offset:32\n\t"
            "global_load_dwordx4 %10, %17, off offset:64\n\t"
            "global_load_dwordx4 %11, %17, off offset:96\n\t"
            "global_load_dwordx4 %12, %17, off offset:128\n\t"
            "global_load_dwordx4 %13, %17, off offset:160\n\t"
            "global_load_dwordx4 %14, %17, off offset:192\n\t"
            "global_load_dwordx4 %15, %17, off offset:224\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3]), "=a"(qf[0][4]),
              "=a"(qf[0][5]), "=a"(qf[0][6]), "=a"(qf[0][7]), "=a"(qf[1][0]), "=a"(qf[1][1]),
              "=a"(qf[1][2]), "=a"(qf[1][3]), "=a"(qf[1][4]), "=a"(qf[1][5]), "=a"(qf[1][6]), "=a"(qf[1][7])
            : "v"(p[0]), "v"(p[1]) : "memory");
    } else if constexpr (KS == 12 && NB == 1) {
        asm volatile(
            "global_load_dwordx4 %0, %12, off\n\t"
            "global_load_dwordx4 %1, %12, off offset:32\n\t"
            "global_load_dwordx4 %2, %12, off offset:64\n\t"
            "global_load_dwordx4 %3, %12, off offset:96\n\t"
            "global_load_dwordx4 %4, %12, off offset:128\n\t"
            "global_load_dwordx4 %5, %12, off offset:160\n\t"
            "global_load_dwordx4 %6, %12, off offset:192\n\t"
            "global_load_dwordx4 %7, %12, off offset:224\n\t"
            "global_load_dwordx4 %8, %12, off offset:256\n\t"
            "global_load_dwordx4 %9, %12, off offset:288\n\t"
            "global_load_dwordx4 %10, %12, off offset:320\n\t"
            "global_load_dwordx4 %11, %12, off offset:352\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3]), "=a"(qf[0][4]),
              "=a"(qf[0][5]), "=a"(qf[0][6]), "=a"(qf[0][7]), "=a"(qf[0][8]), "=a"(qf[0][9]),
              "=a"(qf[0][10]), "=a"(qf[0][11])
            : "v"(p[0]) : "memory");
    } else if constexpr (KS == 12 && NB == 2) {
        asm volatile(
            "global_load_dwordx4 %0, %24, off\n\t"
            "global_load_dwordx4 %1, %24, off offset:32\n\t"
            "global_load_dwordx4 %2, %24, off offset:64\n\t"
            "global_load_dwordx4 %3, %24, off offset:96\n\t"
            "global_load_dwordx4 %4, %24, off offset:128\n\t"
            "global_load_dwordx4 %5, %24, off offset:160\n\t"
            "global_load_dwordx4 %6, %24, off offset:192\n\t"
            "global_load_dwordx4 %7, %24, off offset:224\n\t"
            "global_load_dwordx4 %8, %24, off offset:256\n\t"
            "global_load_dwordx4 %9, %24, off offset:288\n\t"
            "global_load_dwordx4 %10, %24, off offset:320\n\t"
            "global_load_dwordx4 %11, %24, off offset:352\n\t"
            "global_load_dwordx4 %12, %25, off\n\t"
            "global_load_dwordx4 %13, %25, off offset:32\n\t"
            "global_load_dwordx4 %14, %25, off offset:64\n\t"
            "global_load_dwordx4 %15, %25, off offset:96\n\t"
            "global_load_dwordx4 %16, %25, off offset:128\n\t"
            "global_load_dwordx4 %17, %25, off offset:160\n\t"
            "global_load_dwordx4 %18, %25, off offset:192\n\t"
            "global_load_dwordx4 %19, %25, off offset:224\n\t"
            "global_load_dwordx4 %20, %25, off offset:256\n\t"
            "global_load_dwordx4 %21, %25, off offset:288\n\t"
            "global_load_dwordx4 %22, %25, off offset:320\n\t"
            "global_load_dwordx4 %23, %25, off offset:352\n\t"
            "s_waitcnt vmcnt(0)"
            : "=a"(qf[0][0]), "=a"(qf[0][1]), "=a"(qf[0][2]), "=a"(qf[0][3]), "=a"(qf[0][4]),
              "=a"(qf[0][5]), "=a"(qf[0][6]), "=a"(qf[0][7]), "=a"(qf[0][8]), "=a"(qf[0][9]),
              "=a"(qf[0][10]), "=a"(qf[0][11]), "=a"(qf[1][0]), "=a"(qf[1][1]), "=a"(qf[1][2]),
              "=a"(qf[1][3]), "=a"(qf[1][4]), "=a"(qf[1][5]), "=a"(qf[1][6]), "=a"(qf[1][7]),
              "=a"(qf[1][8]), "=a"(qf[1][9]), "=a"(qf[1][10]), "=a"(qf[1][11])
            : "v"(p[0]), "v"(p[1]) : "memory");
    }
}

// o *= alpha for one 16-AGPR accumulator tile, in place, through a single
// temporary VGPR (the accumulators never get a VGPR home).
__device__ __forceinline__ void scale_agpr_tile(f32x16& o, float alpha) {
    float e0 = o[0], e1 = o[1], e2 = o[2], e3 = o[3], e4 = o[4], e5 = o[5], e6 = o[6], e7 = o[7];
    float e8 = o[8], e9 = o[9], e10 = o[10], e11 = o[11], e12 = o[12], e13 = o[13], e14 = o[14], e15 = o[15];
    float tmp;
#define SCALE_ONE(n) "v_accvgpr_read_b32 %16, %" #n "\n\ts_nop 1\n\tv_mul_f32 %16, %16, %17\n\ts_nop 1\n\tv_accvgpr_write_b32 %" #n ", %16\n\t"
    asm volatile(SCALE_ONE(0) SCALE_ONE(1) SCALE_ONE(2) SCALE_ONE(3) SCALE_ONE(4) SCALE_ONE(5) SCALE_ONE(6)
                 SCALE_ONE(7) SCALE_ONE(8) SCALE_ONE(9) SCALE_ONE(10) SCALE_ONE(11) SCALE_ONE(12) SCALE_ONE(13)
                 SCALE_ONE(14) SCALE_ONE(15) "s_nop 1"
                 : "+a"(e0), "+a"(e1), "+a"(e2), "+a"(e3), "+a"(e4), "+a"(e5), "+a"(e6), "+a"(e7), "+a"(e8),
                   "+a"(e9), "+a"(e10), "+a"(e11), "+a"(e12), "+a"(e13), "+a"(e14), "+a"(e15), "=&v"(tmp)
                 : "v"(alpha));
#undef SCALE_ONE
    o[0] = e0; o[1] = e1; o[2] = e2; o[3] = e3; o[4] = e4; o[5] = e5; o[6] = e6; o[7] = e7;
    o[8] = e8; o[9] = e9; o[10] = e10; o[11] = e11; o[12] = e12; o[13] = e13; o[14] = e14; o[15] = e15;
}

template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl<N>(f, std::make_integer_sequence<int, N>());
}
// f(A0), f(A0 + 1), ..., f(A1 - 1)
template <int A0, typename F, int... I>
__device__ __forceinline__ void static_range_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, A0 + I>()), ...);
}
template <int A0, int A1, typename F>
__device__ __forceinline__ void static_range(F&& f) {
    static_range_impl<A0>(f, std::make_integer_sequence<int, A1 - A0>());
}

// NB = 2: 64 query rows per wave, one workgroup (4 waves) per CU. NB = 1: 32
// rows per wave and half the registers, so two workgroups share a CU and each
// SIMD interleaves two waves' instruction streams.
// KVM: the cache layout. KV_CONTIG: K [rows][Hkv][dqk] and V [rows][Hkv][dv];
// KV_PAGED: the same rows in pages reached through a block table; KV_ROPE
// (dqk = 192 only): K split into a per-head part k_nope [rows][Hkv][128] and a
// part shared by all heads k_rope [rows][64], the key layout of the MLA models.
template <int DQK, int DV, int NB, int KVM, bool NT>
__global__ __attribute__((amdgpu_flat_work_group_size(NTHREADS, NTHREADS), amdgpu_waves_per_eu(3 - NB, 3 - NB)))
void attn_fwd_kernel(AttnArgs args, GroupTable) {
    constexpr bool PAGED = KVM == KV_PAGED;
    constexpr bool ROPE = KVM == KV_ROPE;
    static_assert(!ROPE || DQK == 192, "the split key layout is 128 + 64 dims");
    typedef Tiles<DQK, DV, NB> T;
    typedef Atoms<NB> A;
    constexpr int KS = T::KS;
    constexpr int DB = T::DB;
    constexpr int WROWS = 32 * NB;  // query rows per wave
    // LDS fragment prefetch distances (in fragments) of the K and V^T operands; shorter
    // where the 256 registers of a 32-row wave would not hold them beside 192 dims
    constexpr int K_AHEAD = NB == 1 && DQK == 192 ? 2 : 3;
    constexpr int V_AHEAD = NB == 1 && DQK == 192 ? 1 : 2;
    typedef Schedule<T::NQK, T::NPV, DB, NB> SchedFull;
    typedef Schedule<0, T::NPV, DB, NB> SchedLast;
    static_assert(SchedFull().valid() && SchedLast().valid(), "tile schedule breaks a dependency");
    static_assert(SchedFull().qk_tail() >= 4, "the next step's softmax could read S^T before it lands");

    __shared__ __attribute__((aligned(1024))) char smem[T::BYTES];
    char* const kbuf0 = smem;
    char* const vbuf0 = smem + 2 * T::K_BYTES;

    // this workgroup's launch group; the inline table follows the first argument
    auto group_base = [](const LaunchGroup* table) {
        return table ? (uint64_t)(uintptr_t)table
                     : (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(AttnArgs);
    };
    const int gidx0 = find_entry(group_base(args.groups), sizeof(LaunchGroup), args.num_groups, (int)blockIdx.x);
    // A slot holds up to two tiles of the segment: the first runs its key range
    // ascending, its partner from the other end (if any) descending.
#pragma nounroll
    for (int sub = 0; sub < 2; ++sub) {
        // Everything about the tile is worked out again for the second one, from the
        // kernel arguments on (the empty asm hides that it was known), so none of it
        // occupies scalar registers across the key loop.
        int gidx = gidx0;
        const_args_t* ap = (const_args_t*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(gidx), "+s"(ap));
        const_args_t& a = *ap;
        const_group_t* const grp = const_ptr<const_group_t>(group_base(a.groups)) + gidx;
        // read at once (the empty asm needs them all here): left to the compiler, each is
        // read where it is first used, five latencies in a row
        LaunchGroup g{grp->wg0, grp->row0, grp->len, grp->prefix, grp->kv_start, grp->seg, grp->pieces, grp->part0, grp->slots, grp->tiles};
        TileArgs ta{a.group, a.pack, a.tile_tokens, a.head_groups, a.xcd_remap};
        asm volatile("" : "+s"(g.wg0), "+s"(g.row0), "+s"(g.len), "+s"(g.prefix), "+s"(g.kv_start), "+s"(g.pieces), "+s"(g.part0),
                          "+s"(g.slots), "+s"(g.tiles), "+s"(ta.group), "+s"(ta.pack), "+s"(ta.tile_tokens),
                          "+s"(ta.head_groups), "+s"(ta.xcd_remap));
        TileWork it;
        if (!tile_work(ta, g, (int)blockIdx.x - g.wg0, sub, it)) break;
        const int h = it.h, hk = it.hk, out_row0 = it.out_row0;
        const int64_t kv_start = g.kv_start;
        // every wave is done with the LDS tiles of the slot's previous tile before
        // this tile's first copies overwrite them
        lds_barrier();
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // nor any lane's offsets vector registers
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS bases stay scalar
        const int lr = lane & 31;
        const int lg = lane >> 5;

        const int kb = it.key_begin, ke = it.key_end;
        // contiguous cache: the request's row 0 of head hk; paged: page 0's row 0
        const int64_t cache_row0 = PAGED ? 0 : kv_start;
        const u16* kbase = a.k + cache_row0 * a.k_st + (int64_t)hk * a.k_sh;
        const u16* vbase = a.v + cache_row0 * a.v_st + (int64_t)hk * a.v_sh;
        const int ntiles = (ke - kb + BN - 1) / BN;
        // key tiles sit at kb + m*BN (m = 0 .. ntiles-1) in both directions; visit j
        // of the tile loop reads the tile at kt_first + j*dkt
        const bool rev = sub != 0;
        const int dkt = rev ? -BN : BN;
        const int kt_first = rev ? kb + (ntiles - 1) * BN : kb;
        // paged cache: this segment's block-table row and the cache row of key 0
        const int32_t* bt_row = PAGED ? a.block_table + (int64_t)g.seg * a.bt_st : nullptr;
        const int kv_off = PAGED ? (int)kv_start : 0;
        const int pmask = PAGED ? (1 << a.page_shift) - 1 : 0;
        const int last_row = kv_off + ke - 1;  // page reads past the key range are clamped here
        auto clamp_page = [&](int pg) { return (int)min((uint32_t)pg, (uint32_t)(a.num_pages - 1)); };
        auto page_of = [&](int row) {  // synchronous lookup (prologue)
            return clamp_page(__builtin_amdgcn_readfirstlane(bt_row[min(row, last_row) >> a.page_shift]));
        };
        // first element of the tile of keys starting at kt
        auto tile_src = [&](const u16* base, int64_t page_st, int64_t row_st, int kt) -> const u16* {
            if constexpr (PAGED) {
                const int row = kv_off + kt;
                return base + (int64_t)page_of(row) * page_st + (int64_t)(row & pmask) * row_st;
            } else {
                return base + (int64_t)kt * row_st;
            }
        };

        // This lane's NB query rows (one per 32-column block of S^T), as B
        // operands in AGPRs. Rows past the tile re-read its last row (their results
        // are never stored), so every load stays inside q.
        const int tile_rows = it.nrows * a.pack;  // at most BM
        bf16x8 qf[NB][KS];
        const u16* qp[NB];
        int qlim[NB];   // last key position the row may see, minus lg*4 (see masking)
        bool qvalid[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int rloc = wave * WROWS + nb * 32 + lr;
            qvalid[nb] = rloc < tile_rows;
            const int r = min(rloc, tile_rows - 1);
            const int tok = row_token(r, a.pack_magic);
            qlim[nb] = min(it.pos0 + tok, ke - 1) - lg * 4;
            qp[nb] = a.q + (int64_t)(it.row0 + tok) * a.q_st + (int64_t)(h + r - tok * a.pack) * a.q_sh + lg * 8;
        }
        const int wave_first = it.pos0 + row_token(wave * WROWS, a.pack_magic);

        // Global->LDS copy of one tile through a buffer resource whose base is the
        // tile's first key row and whose size ends at the last key of the range:
        // rows past the range read as zeros (buffer range check), so the last tile
        // needs no special case. Per-lane byte offsets are fixed for the kernel.
        // Split key layout: the K tile is two LDS regions, the per-head part
        // [BN][NOPE_GR] granules then the shared part [BN][ROPE_GR], each filled by
        // its own copies (a copy instruction has one source) and swizzled for its
        // own row width; the first NOPE_LOADS copies read k_nope, the rest k_rope.
        constexpr int NOPE_LOADS = BN * NOPE_GR / NTHREADS;
        constexpr int NOPE_BYTES = BN * NOPE_GR * 16;
        uint32_t k_src[T::K_LOADS], v_src[T::V_LOADS];
#pragma unroll
        for (int t = 0; t < T::K_LOADS; ++t) {
            if constexpr (ROPE) {
                if (t < NOPE_LOADS) {
                    const int slot = t * NTHREADS + tid;
                    const int row = slot / NOPE_GR, gs = slot % NOPE_GR;
                    k_src[t] = (uint32_t)(row * (int)a.k_st + kswz<NOPE_GR>(row, gs) * 8) * 2u;
                } else {
                    const int slot = (t - NOPE_LOADS) * NTHREADS + tid;
                    const int row = slot / ROPE_GR, gs = slot % ROPE_GR;
                    k_src[t] = (uint32_t)(row * (int)a.kr_st + kswz<ROPE_GR>(row, gs) * 8) * 2u;
                }
            } else {
                const int slot = t * NTHREADS + tid;
                const int row = slot / T::KGR, gs = slot % T::KGR;
                k_src[t] = (uint32_t)(row * (int)a.k_st + kswz<T::KGR>(row, gs) * 8) * 2u;
            }
        }
#pragma unroll
        for (int t = 0; t < T::V_LOADS; ++t) {
            const int slot = t * NTHREADS + tid;
            const int row = slot / T::VGR, gs = slot % T::VGR;
            v_src[t] = (uint32_t)(row * (int)a.v_st + vswz<T::VGR>(row, gs) * 8) * 2u;
        }
        // resources over the rows [kt, min(kt + BN, ke)) (none when kt >= ke); the host
        // keeps row strides below 2^31 / (2 BN) elements, so a tile's byte count fits
        auto tile_bytes = [&](int kt, int32_t row_st) {
            return (int32_t)((uint32_t)max(0, min(BN, ke - kt)) * (uint32_t)row_st * 2u);
        };
        auto k_rsrc = [&](int kt) { return make_rsrc(tile_src(kbase, a.k_sp, a.k_st, kt), tile_bytes(kt, a.k_st)); };
        // the shared key part of the same rows (split layout; one row per key, no head)
        const u16* rbase = ROPE ? a.k_rope + cache_row0 * a.kr_st : nullptr;
        auto kr_rsrc = [&](int kt) { return make_rsrc(rbase + (int64_t)kt * a.kr_st, tile_bytes(kt, a.kr_st)); };
        auto v_rsrc = [&](int kt) { return make_rsrc(tile_src(vbase, a.v_sp, a.v_st, kt), tile_bytes(kt, a.v_st)); };
        const uint32_t lds_wave = (uint32_t)(uintptr_t)(lds_void_t*)smem + (uint32_t)wave * 1024u;
        // copy t of the K (V) tile into buffer B: LDS offset from this wave's base
        auto load_k = [&](const i32x4& r, const i32x4& rr, auto B, auto TT) {
            constexpr int t = decltype(TT)::value;
            if constexpr (ROPE && t >= NOPE_LOADS) {
                constexpr int off = decltype(B)::value * T::K_BYTES + NOPE_BYTES + (t - NOPE_LOADS) * NWAVES * 1024;
                copy16_to_lds<off, NT>(rr, lds_wave, k_src[t]);
            } else {
                constexpr int off = decltype(B)::value * T::K_BYTES + t * NWAVES * 1024;
                copy16_to_lds<off, NT>(r, lds_wave, k_src[t]);
            }
        };
        auto load_v = [&](const i32x4& r, auto B, auto TT) {
            constexpr int off = 2 * T::K_BYTES + decltype(B)::value * T::V_BYTES + decltype(TT)::value * NWAVES * 1024;
            copy16_to_lds<off, NT>(r, lds_wave, v_src[decltype(TT)::value]);
        };
        auto issue_k = [&](auto B, int kt) {
            const i32x4 r = k_rsrc(kt);
            const i32x4 rr = ROPE ? kr_rsrc(kt) : r;
            static_for<T::K_LOADS>([&](auto TT) { load_k(r, rr, B, TT); });
        };
        auto issue_v = [&](auto B, int kt) {
            const i32x4 r = v_rsrc(kt);
            static_for<T::V_LOADS>([&](auto TT) { load_v(r, B, TT); });
        };
        if (ntiles > 0) {
            issue_k(std::integral_constant<int, 0>(), kt_first);
            issue_v(std::integral_constant<int, 0>(), kt_first);
            if (ntiles > 1) issue_k(std::integral_constant<int, 1>(), kt_first + dkt);
        }
        // The query rows travel with the first copies: one latency (4 to 5 thousand
        // cycles on a busy chip) where Q first and then the copies cost 1.5 to 2
        // thousand more.
        load_q_agpr<KS, NB>(qf, qp);

        // Per-lane LDS byte offsets; the rest of each address is an immediate.
        // K (A operand of S^T): row mb*32+lr, logical granule ks*2+lg; row & 15 and
        // (row >> 1) & 7 depend only on lr. The swizzle touches the low 4 (or 3)
        // bits of the granule index, so K_OFFS offsets cover every ks and the
        // higher granule bits are an immediate.
        // (split key layout: K_OFFS offsets for the per-head region, KR_OFFS for the
        // shared one)
        constexpr int K_OFFS = ROPE ? NOPE_GR / 2 : ((T::KGR % 16 == 0) ? 8 : 4);
        constexpr int KR_OFFS = ROPE ? ROPE_GR / 2 : 1;
        int k_off[K_OFFS], kr_off[KR_OFFS];
#pragma unroll
        for (int r = 0; r < K_OFFS; ++r) {
            if constexpr (ROPE) k_off[r] = lr * (NOPE_GR * 16) + kswz<NOPE_GR>(lr, r * 2 + lg) * 16;
            else k_off[r] = lr * (T::KGR * 16) + kswz<T::KGR>(lr, r * 2 + lg) * 16;
        }
#pragma unroll
        for (int r = 0; r < KR_OFFS; ++r) kr_off[r] = ROPE ? lr * (ROPE_GR * 16) + kswz<ROPE_GR>(lr, r * 2 + lg) * 16 : 0;
        // V^T (A operand of O^T) through ds_read_b64_tr_b16: 16-lane group q reads
        // keys 4*(q>>1) + (j>>2) and value columns 16*(q&1) + 4*(j&3) .. +3, i.e.
        // granule 4*d + (tr_col >> 3) of value block d; key & 3 = tr_key & 3.
        const int tq = lane >> 4, tj = lane & 15;
        const int tr_key = 4 * (tq >> 1) + (tj >> 2);
        const int tr_col = 16 * (tq & 1) + 4 * (tj & 3);
        // The LDS offset of the V buffers is part of the register (the empty asm keeps it
        // there): added to an immediate it would pass the 16 bits of one at dqk = 192.
        uint32_t v_off[DB];
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            v_off[d] = (uint32_t)(uintptr_t)(lds_void_t*)vbuf0 + tr_key * (T::VGR * 16) +
                       vswz<T::VGR>(tr_key, d * 4 + (tr_col >> 3)) * 16 + (tr_col & 7) * 2;
            asm volatile("" : "+v"(v_off[d]));
        }

        float m_run[NB];   // max used by exp2 (log2 units), refreshed lazily
        float l_part[NB];  // this lane's share of the softmax denominator
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            m_run[nb] = -INFINITY;
            l_part[nb] = 0.f;
        }
        f32x16 o[DB][NB];
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[d][nb][i] = 0.f;

        auto load_kfrag = [&](const char* kt_buf, int ks, int mb) -> bf16x8 {
            if constexpr (ROPE) {
                const char* addr = ks < NOPE_GR / 2
                                       ? kt_buf + mb * 32 * NOPE_GR * 16 + k_off[ks]
                                       : kt_buf + NOPE_BYTES + mb * 32 * ROPE_GR * 16 + kr_off[ks - NOPE_GR / 2];
                return __builtin_bit_cast(bf16x8, *(const u32x4*)addr);
            } else {
                const u32x4 raw = *(const u32x4*)(kt_buf + mb * 32 * T::KGR * 16 + (ks / K_OFFS) * (K_OFFS * 32) +
                                                  k_off[ks % K_OFFS]);
                return __builtin_bit_cast(bf16x8, raw);
            }
        };
        typedef __attribute__((address_space(3))) char lds_char_t;
        auto load_vfrag = [&](int vt, int mb, int hh, int d) -> bf16x8 {  // vt: byte offset of the V buffer
            bf16x8 af;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                lds_char_t* addr = (lds_char_t*)(uintptr_t)v_off[d] + (vt + (mb * 32 + hh * 16 + half * 8) * T::VGR * 16);
                const i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)addr);
                const bf16x4 rb = __builtin_bit_cast(bf16x4, r);
#pragma unroll
                for (int j = 0; j < 4; ++j) af[half * 4 + j] = rb[j];
            }
            return af;
        };

        // S^T = K Q^T for a whole tile (prologue only: no softmax to overlap with)
        auto qk_all = [&](const char* kt_buf, f32x16 (&s)[2][NB]) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    const bf16x8 af = load_kfrag(kt_buf, ks, mb);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const bf16x8 bq = qf[nb][ks];
                        if (ks == 0) MFMA_32x32x16_INIT(s[mb][nb], af, bq);
                        else MFMA_32x32x16_ACC(s[mb][nb], af, bq);
                    }
                }
        };

        // Running sources of the copies a step issues (K of visit t+2, V of visit
        // t+1): scalar pointer, first key and visits left, advanced by one tile per
        // step. Past the last visit a copy gets an empty resource; its pointer may
        // then run outside the tensor, but an empty resource never reads it.
        const uint32_t k_row_bytes = (uint32_t)a.k_st * 2u, v_row_bytes = (uint32_t)a.v_st * 2u;
        // V of visit t+1 is one visit behind K of visit t+2: its first key is
        // kt_k - dkt and it has one visit more left
        uint64_t k_next = PAGED ? 0 : (uint64_t)(uintptr_t)kbase + (uint64_t)((int64_t)(kt_first + 2 * dkt) * k_row_bytes);
        uint64_t v_next = PAGED ? 0 : (uint64_t)(uintptr_t)vbase + (uint64_t)((int64_t)(kt_first + dkt) * v_row_bytes);
        int kt_k = kt_first + 2 * dkt;
        int k_left = ntiles - 2;
        // split key layout: the shared part's running source (same rows as K)
        const uint32_t kr_row_bytes = ROPE ? (uint32_t)a.kr_st * 2u : 0u;
        uint64_t kr_next = ROPE ? (uint64_t)(uintptr_t)rbase + (uint64_t)((int64_t)(kt_first + 2 * dkt) * kr_row_bytes) : 0;
        // one tile of rows in bytes (below 2^31), signed by the direction
        auto tile_step = [&](uint32_t row_bytes) { return (uint64_t)(int64_t)(rev ? -(int32_t)(BN * row_bytes) : (int32_t)(BN * row_bytes)); };
        // paged cache: the page of the K tile a step copies is read one step ahead
        // (raw, clamped at its use), and V(t+1) shares K(t+1)'s page; table reads
        // are clamped to the rows of the key range
        auto clamp_row = [&](int row) { return min(max(row, kv_off + kb), last_row); };
        int pg_pending = 0, pg_prev = 0;
        if constexpr (PAGED) {
            if (ntiles > 0) {
                pg_prev = page_of(clamp_row(kv_off + kt_first + dkt));
                pg_pending = bt_row[clamp_row(kv_off + kt_first + 2 * dkt) >> a.page_shift];
            }
        }

        float scale_log2 = a.scale_log2;
        asm volatile("" : "+s"(scale_log2));  // held in a register, not read again every step

        // One key tile: mask S(t) if needed, then the scheduled mix of S(t+1)
        // MFMAs, the softmax of S(t) and the O^T += V^T P^T MFMAs of tile t.
        auto step = [&](auto P, auto HAS_NEXT, int t, f32x16 (&s_cur)[2][NB], f32x16 (&s_nxt)[2][NB]) {
            constexpr int par = decltype(P)::value;
            constexpr bool has_next = decltype(HAS_NEXT)::value;
            const char* kt_nxt = kbuf0 + (1 - par) * T::K_BYTES;
            constexpr int vt_cur = par * T::V_BYTES;
            const int kt = kt_first + t * dkt;
            wait_vmcnt<0>();
            lds_barrier();  // K(t+1), V(t) are in LDS; every wave is done with K(t) and V(t-1)
            // the next tiles' copies (K(t+2) into the K buffer just freed, V(t+1)
            // into the V buffer just freed) are spread over the first slots. Past
            // the last tile the resources are empty: the copies then only write
            // zeros into buffers that no later step reads, and the step needs no
            // branch around them.
            if constexpr (PAGED) {
                // the page read during the previous step is complete after the
                // barrier; the empty asm pins its use here, before any LDS read of
                // this step is in flight
                int pg_k = clamp_page(__builtin_amdgcn_readfirstlane(pg_pending));
                asm volatile("" : "+s"(pg_k) : : "memory");
                const int row_k = kv_off + kt_k, row_v = row_k - dkt;
                k_next = (uint64_t)(uintptr_t)(kbase + (int64_t)pg_k * a.k_sp + (int64_t)(row_k & pmask) * a.k_st);
                v_next = (uint64_t)(uintptr_t)(vbase + (int64_t)pg_prev * a.v_sp + (int64_t)(row_v & pmask) * a.v_st);
                pg_prev = pg_k;
                pg_pending = bt_row[clamp_row(row_k + dkt) >> a.page_shift];
            }
            // rows of the copied tile (a tile is partial only at the end of the
            // range), times the row bytes (below 2^31); none past the last visit
            const uint32_t k_n = k_left > 0 ? (uint32_t)min(BN, ke - kt_k) : 0u;
            const uint32_t v_n = k_left >= 0 ? (uint32_t)min(BN, ke - (kt_k - dkt)) : 0u;
            const i32x4 rk = make_rsrc((const void*)k_next, (int32_t)(k_n * k_row_bytes));
            const i32x4 rv = make_rsrc((const void*)v_next, (int32_t)(v_n * v_row_bytes));
            i32x4 rkr = rk;
            if constexpr (ROPE) {
                rkr = make_rsrc((const void*)kr_next, (int32_t)(k_n * kr_row_bytes));
                kr_next += tile_step(kr_row_bytes);
            }
            if constexpr (!PAGED) {
                k_next += tile_step(k_row_bytes);
                v_next += tile_step(v_row_bytes);
            }
            kt_k += dkt;
            --k_left;

            // causal / range mask on the tiles that cross a row's last visible key:
            // key kt + c (c = mb*32 + (i>>2)*8 + lg*4 + (i&3)) is hidden when
            // c > qlim - kt, with qlim = min(row position, ke - 1) - lg*4
            if ((kt + BN - 1 > wave_first) || (kt + BN > ke)) {
                const float ninf = -INFINITY;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int lim = qlim[nb] - kt;
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            // compare and select through VCC, one element at a time (no
                            // batch of 64-bit lane masks in scalar registers)
                            float x = s_cur[mb][nb][i];
                            asm("v_cmp_gt_i32 vcc, %2, %1\n\tv_cndmask_b32 %0, %0, %3, vcc"
                                : "+v"(x)
                                : "v"(lim), "i"(mb * 32 + (i >> 2) * 8 + (i & 3)), "v"(ninf)
                                : "vcc");
                            s_cur[mb][nb][i] = x;
                        }
                }
            }

            float alpha[NB], m_use[NB], mx[NB][4], lsum[NB][2];  // mx: one partial max per max atom
            bool refresh[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                alpha[nb] = 1.f;
                m_use[nb] = 0.f;
                lsum[nb][0] = lsum[nb][1] = 0.f;
                refresh[nb] = false;
            }
            float pprev = 0.f;
            bf16x8 pb[NB][2][2];         // [nb][mb][hh]
            bf16x8 kf[K_AHEAD + 1];      // K fragments in issue order, K_AHEAD in flight
            bf16x8 vf[V_AHEAD + 1];      // V^T fragments in issue order, V_AHEAD in flight

            auto atom = [&](auto K) {
                constexpr int k = decltype(K)::value;
                if constexpr (k < A::MAXF) {
                    // max of 8 of the 32 scores of query block nb, as a depth-2 tree:
                    // the four atoms of a row are independent of each other
                    constexpr int nb = k >> 2, q = k & 3;
                    auto sc = [&](int j) -> float {
                        const int v = q * 8 + j;  // score index in [mb*16 + i]
                        return s_cur[v >> 4][nb][v & 15];
                    };
                    const float t0 = max3f(sc(0), sc(1), sc(2));
                    const float t1 = max3f(sc(3), sc(4), sc(5));
                    const float t2 = max2f(sc(6), sc(7));
                    mx[nb][q] = max3f(t0, t1, t2);
                } else if constexpr (k < A::EXP) {
                    constexpr int nb = k - A::MAXF;
                    const float m =
                        lane_swap32_max(max3f(mx[nb][0], mx[nb][1], max2f(mx[nb][2], mx[nb][3]))) * scale_log2;
                    // per-lane decision: the exps of this row wait only for VALU work;
                    // the wave-wide vote happens once, at the rescale check
                    refresh[nb] = m > m_run[nb] + LAZY_TAU;
                    const float m_new = refresh[nb] ? m : m_run[nb];
                    // a row that has seen no visible key yet (m_new = -inf) has nothing to rescale
                    alpha[nb] = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_run[nb] - m_new);
                    m_run[nb] = m_new;
                    m_use[nb] = (m_new == -INFINITY) ? 0.f : m_new;
                    l_part[nb] *= alpha[nb];
                } else {
                    constexpr int e = k - A::EXP;
                    constexpr int u = e >> 3, j = e & 7;
                    constexpr int mb = u / (2 * NB), hh = (u / NB) & 1, nb = u % NB;
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[mb][nb][hh * 8 + j], scale_log2, -m_use[nb]));
                    lsum[nb][j & 1] += pv;
                    if constexpr ((j & 1) == 0) {
                        pprev = pv;
                    } else {
                        pb[nb][mb][hh][j - 1] = (__bf16)pprev;
                        pb[nb][mb][hh][j] = (__bf16)pv;
                    }
                }
            };

            auto run = [&](auto tag) {
                typedef typename decltype(tag)::type Sch;
                constexpr Sch sch{};
                constexpr int NS = Sch::NS;
                typedef QkCoords<KS, NB> C;
                // fragments needed first: V_AHEAD V^T fragments, and K_AHEAD K fragments of the next tile
                static_for<V_AHEAD>([&](auto I) {
                    constexpr int f = I;
                    vf[f] = load_vfrag(vt_cur, (f / DB) >> 1, (f / DB) & 1, f % DB);
                });
                if constexpr (has_next)
                    static_for<K_AHEAD>([&](auto I) {
                        constexpr int f = I;
                        kf[f] = load_kfrag(kt_nxt, C::ks(NB * f), C::mb(NB * f));
                    });
                static_for<NS>([&](auto SL) {
                    constexpr int s = SL;
                    constexpr int kind = sch.kind[s];
                    constexpr int idx = sch.index[s];
                    if constexpr (s == sch.rescale_before) {
                        bool any = false;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) any = any || refresh[nb];
                        // nothing to rescale on the first tile: O is zero
                        if (t > 0 && __builtin_amdgcn_ballot_w64(any) != 0) {
                            // rare: rescale the AGPR accumulators 16 at a time, so the
                            // branch needs only a few temporary VGPRs (alpha = 1 in the
                            // lanes whose reference did not move)
                            mfma_drain();
                            static_for<NB * DB>([&](auto J) {
                                constexpr int nb = J / DB, d = J % DB;
                                scale_agpr_tile(o[d][nb], alpha[nb]);
                                __builtin_amdgcn_sched_barrier(0);
                            });
                        }
                    }
                    if constexpr (has_next) {
                        constexpr int NL = T::K_LOADS + T::V_LOADS;
                        constexpr int LSTRIDE = (NS / LOAD_SPREAD) / NL > 0 ? (NS / LOAD_SPREAD) / NL : 1;
                        if constexpr (s % LSTRIDE == 0 && s / LSTRIDE < NL) {
                            constexpr int j = s / LSTRIDE;
                            if constexpr (j < T::V_LOADS) {
                                load_v(rv, std::integral_constant<int, 1 - par>(), std::integral_constant<int, j>());
                            } else {
                                load_k(rk, rkr, std::integral_constant<int, par>(),
                                       std::integral_constant<int, j - T::V_LOADS>());
                            }
                        }
                    }
                    if constexpr (kind == 2) {
                        // VALU-only slot
                    } else if constexpr (kind == 0) {
                        constexpr int ks = C::ks(idx), mb = C::mb(idx), nb = C::nb(idx);
                        constexpr int frag = idx / NB;  // (mb, ks) in issue order
                        // prefetch K_AHEAD fragments ahead with this fragment's first MFMA
                        if constexpr (nb == 0 && frag + K_AHEAD < 2 * KS)
                            kf[(frag + K_AHEAD) % (K_AHEAD + 1)] =
                                load_kfrag(kt_nxt, C::ks(NB * (frag + K_AHEAD)), C::mb(NB * (frag + K_AHEAD)));
                        const bf16x8 af = kf[frag % (K_AHEAD + 1)];
                        const bf16x8 bq = qf[nb][ks];
                        if constexpr (ks == 0) MFMA_32x32x16_INIT(s_nxt[mb][nb], af, bq);
                        else MFMA_32x32x16_ACC(s_nxt[mb][nb], af, bq);
                    } else {
                        constexpr int grp = idx / (NB * DB), d = (idx / NB) % DB, nb = idx % NB;
                        constexpr int mb = grp >> 1, hh = grp & 1;
                        constexpr int frag = idx / NB;  // (grp, d) in issue order
                        // prefetch V_AHEAD fragments ahead with this fragment's first MFMA
                        if constexpr (nb == 0 && frag + V_AHEAD < 4 * DB) {
                            constexpr int f2 = frag + V_AHEAD;
                            vf[f2 % (V_AHEAD + 1)] = load_vfrag(vt_cur, (f2 / DB) >> 1, (f2 / DB) & 1, f2 % DB);
                        }
                        o[d][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[frag % (V_AHEAD + 1)], pb[nb][mb][hh],
                                                                           o[d][nb], 0, 0, 0);
                    }
                    constexpr int a0 = s == 0 ? 0 : sch.atoms_end[s == 0 ? 0 : s - 1];
                    constexpr int a1 = sch.atoms_end[s];
                    static_range<a0, a1>([&](auto K) { atom(K); });
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            if constexpr (has_next) run(std::type_identity<SchedFull>());
            else run(std::type_identity<SchedLast>());
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) l_part[nb] += lsum[nb][0] + lsum[nb][1];
        };

        if (ntiles > 0) {
            typedef std::integral_constant<int, 0> P0;
            typedef std::integral_constant<int, 1> P1;
            typedef std::integral_constant<bool, true> NX;
            typedef std::integral_constant<bool, false> LAST;
            f32x16 s_a[2][NB], s_b[2][NB];
            lds_barrier();
            qk_all(kbuf0, s_a);
            mfma_drain();
            // Tiles in pairs (static buffer parity). With an even tile count the
            // last pair computes one S^T tile too many, from stale LDS data, and
            // discards it: cheaper than a third step variant's registers.
            int t = 0;
            // Where the loop starts in its 64-byte line of code decides up to 1 % at these
            // sizes (16384 rows behind 507904, 16 MLA heads: 65.6 ms at 16 of 64, 66.5 at 8,
            // 65.9 at 24); two instructions follow before it.
            if constexpr (DQK == 192 && NB == 2) asm volatile(".p2align 6\n\ts_nop 0\n\ts_nop 0");
            for (; t + 1 < ntiles; t += 2) {
                step(P0(), NX(), t, s_a, s_b);
                step(P1(), NX(), t + 1, s_b, s_a);
            }
            if (t < ntiles) step(P0(), LAST(), t, s_a, s_b);
            mfma_drain();
            // a pair's second step may still be copying (zeros) into LDS: no copy
            // may outlive the workgroup's LDS allocation
            wait_vmcnt<0>();
        }

        // ---- epilogue: normalise and store ----
        // The arguments only the epilogue needs are read again from the kernel
        // argument segment (the empty asm hides that they were read before), so
        // they do not occupy scalar registers across the key loop.
        const_args_t* ka = (const_args_t*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ka));
        const bool partial = out_row0 < 0;
        const int row0 = partial ? ~out_row0 : out_row0;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const float l_tot = lane_swap32_add(l_part[nb]);
            const float inv_l = l_tot > 0.f ? 1.f / l_tot : 0.f;
            const float lse_val = l_tot > 0.f ? (m_run[nb] + __log2f(l_tot)) * 0.69314718055994531f : -INFINITY;
            const int rloc = wave * WROWS + nb * 32 + lr;
            const int tok = row_token(rloc, ka->pack_magic);
            const int row = row0 + tok, hh = h + rloc - tok * ka->pack;
            if (partial) {
                if (!qvalid[nb]) continue;
                const int64_t prow = (int64_t)row * ka->num_heads + hh;
                float* po = ka->part_o + prow * DV;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float4 w = {o[d][nb][c * 4 + 0] * inv_l, o[d][nb][c * 4 + 1] * inv_l,
                                    o[d][nb][c * 4 + 2] * inv_l, o[d][nb][c * 4 + 3] * inv_l};
                        *(float4*)(po + d * 32 + c * 8 + lg * 4) = w;
                    }
                if (lg == 0) ka->part_lse[prow] = lse_val;
            } else {
                // A lane holds columns c*8 + lg*4 .. +3 of its row, its partner (lane ^ 32)
                // the other four of each eight: for two values of c they exchange halves, and
                // each stores 16 bytes. Stores of 8 bytes took twice as many instructions, each
                // touching as many lines.
                u16* op = ka->out + (int64_t)row * ka->o_st + (int64_t)hh * ka->o_sh + lg * 8;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int c = 0; c < 4; c += 2) {
                        u32x2 w[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            bf16x4 x;
#pragma unroll
                            for (int j = 0; j < 4; ++j) x[j] = (__bf16)(o[d][nb][(c + e) * 4 + j] * inv_l);
                            w[e] = __builtin_bit_cast(u32x2, x);
                        }
                        const auto lo = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                        const auto hi = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                        const u32x4 v = {lo[0], hi[0], lo[1], hi[1]};
                        if (qvalid[nb]) *(u32x4*)(op + d * 32 + c * 8) = v;
                    }
                if (lg == 0 && qvalid[nb] && ka->lse) ka->lse[(int64_t)hh * ka->lse_sh + row] = lse_val;
            }
        }
    }  // slot tiles
}


// Lane groups that share the pieces of one (row, head) in the merge. Many pieces
// mean few rows (a split is what fills the chip with them), and one group walking 37
// pieces takes 14 us of load latency: up to eight take every eighth piece each.
__host__ __device__ constexpr int merge_ways(int pieces) {
    return pieces >= 16 ? 8 : pieces >= 8 ? 4 : pieces >= 4 ? 2 : 1;
}

// (row, head) pair of a segment -- of its len * num_heads in that order -- that lane group
// `grp` of `groups` merges in the segment's block `block`; `way`: the pieces it takes,
// every ways-th from `way` on. Past the last pair: none.
__host__ __device__ __forceinline__ int64_t merge_place(int block, int groups, int grp, int ways, int& way) {
    way = grp % ways;
    return (int64_t)block * (groups / ways) + grp / ways;
}

// Merge of split partials: lse = log sum_b exp(lse_b); out = sum_b exp(lse_b - lse) O_b.
// DV/4 threads a lane group, 4 values each; a block stays within one segment.
template <int DV>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a, CombineTable) {
    constexpr int G = DV / 4, GROUPS = 256 / G;
    const uint64_t table = a.segs ? (uint64_t)(uintptr_t)a.segs
                                  : (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(CombineArgs);
    const_seg_t* const sg = const_ptr<const_seg_t>(table) +
                            find_entry(table, sizeof(CombineSeg), a.num_segs, (int)blockIdx.x);
    const int len = sg->len, n = sg->pieces;
    const int ways = merge_ways(n);
    const int grp = threadIdx.x / G, c = threadIdx.x % G;
    int way;
    const int64_t pairs = (int64_t)len * a.num_heads;
    const int64_t pair = merge_place((int)blockIdx.x - sg->block0, GROUPS, grp, ways, way);
    const bool valid = pair < pairs;
    const int64_t at = valid ? pair : pairs - 1;  // spare groups repeat the last pair, and store nothing
    const int row = (int)(at / a.num_heads);
    const int h = (int)(at - (int64_t)row * a.num_heads);
    // piece b of the pair: `pairs` entries further on
    const float* const pl = a.part_lse + (int64_t)sg->part0 * a.num_heads + at;
    const float* const po = a.part_o + ((int64_t)sg->part0 * a.num_heads + at) * DV + c * 4;
    float mx = -INFINITY, den = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    // Four pieces in flight. Past the last one: weight 0, and zeros, nothing being read there
    // (0 times an infinite partial would be NaN; reading piece b0 again cost 2 to 4 us a call,
    // 1500 rows of 16 heads behind 16000 keys in 8 pieces 245.3 and 241.9).
    auto four = [&](int b0, auto whole) {
        float l[4];
        float4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t b = b0 + j * ways;
            l[j] = -INFINITY;
            v[j] = {0.f, 0.f, 0.f, 0.f};
            if (whole || b < n) {
                l[j] = pl[b * pairs];
                v[j] = *(const float4*)(po + b * pairs * DV);
            }
        }
        const float m = fmaxf(mx, fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
        const float keep = mx == -INFINITY ? 0.f : __expf(mx - m);
        den *= keep;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] *= keep;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float w = l[j] == -INFINITY ? 0.f : __expf(l[j] - m);
            den += w;
            acc[0] += w * v[j].x;
            acc[1] += w * v[j].y;
            acc[2] += w * v[j].z;
            acc[3] += w * v[j].w;
        }
        mx = m;
    };
    int first = 0;  // the same in all lane groups of a row: a wave takes one of the two
    for (; first + 4 * ways <= n; first += 4 * ways) four(first + way, std::true_type());
    if (first < n) four(first + way, std::false_type());
    if (ways > 1) {  // the block's segment decides: uniform
        __shared__ float4 s_acc[256];
        __shared__ float2 s_md[GROUPS];
        s_acc[threadIdx.x] = {acc[0], acc[1], acc[2], acc[3]};
        if (c == 0) s_md[grp] = {mx, den};
        __syncthreads();
        if (way != 0) return;
        float m = mx;
        for (int w = 1; w < ways; ++w) m = fmaxf(m, s_md[grp + w].x);
        const float keep = mx == -INFINITY ? 0.f : __expf(mx - m);
        den *= keep;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] *= keep;
        for (int w = 1; w < ways; ++w) {
            const float2 md = s_md[grp + w];
            const float4 v = s_acc[threadIdx.x + w * G];
            const float f = md.x == -INFINITY ? 0.f : __expf(md.x - m);
            den += f * md.y;
            acc[0] += f * v.x;
            acc[1] += f * v.y;
            acc[2] += f * v.z;
            acc[3] += f * v.w;
        }
        mx = m;
    }
    if (!valid) return;
    const float inv = den > 0.f ? 1.f / den : 0.f;  // no visible key has any weight: zeros, as without a split
    bf16x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = (__bf16)(acc[j] * inv);
    const int64_t orow = (int64_t)sg->row0 + row;
    *(bf16x4*)(a.out + orow * a.o_st + (int64_t)h * a.o_sh + c * 4) = r;
    if (c == 0 && a.lse) a.lse[(int64_t)h * a.lse_sh + orow] = mx + __logf(den);
}

[[maybe_unused]] size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

template <int DQK, int DV, int NB, int KVM, bool NT>
hipError_t launch_kernels(const Launch& l, hipStream_t stream) {
    if (l.workgroups <= 0) return hipSuccess;
    if (l.workgroups > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((attn_fwd_kernel<DQK, DV, NB, KVM, NT>), dim3((unsigned)l.workgroups), dim3(NTHREADS), 0, stream,
                       l.a, l.groups);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || l.merge.blocks == 0) return e;
    hipLaunchKernelGGL((combine_kernel<DV>), dim3((unsigned)l.merge.blocks), dim3(256), 0, stream, l.merge, l.segs);
    return hipGetLastError();
}

template <int DQK, int DV, int NB, int KVM>
hipError_t launch(const Launch& l, hipStream_t stream) {
    if constexpr (NB == 1)
        if (l.nt) return launch_kernels<DQK, DV, NB, KVM, true>(l, stream);
    return launch_kernels<DQK, DV, NB, KVM, false>(l, stream);
}

template <int KVM>
hipError_t launch_dims(const Launch& l, hipStream_t stream) {
    if constexpr (KVM == KV_ROPE) {
        // the split key layout exists for dqk = 192 only (the caller checks)
        if (l.nb == 1) return launch<192, 128, 1, KVM>(l, stream);
        return launch<192, 128, 2, KVM>(l, stream);
    } else {
        if (l.nb == 1) {
            if (l.dqk == 64) return launch<64, 64, 1, KVM>(l, stream);
            if (l.dqk == 128) return launch<128, 128, 1, KVM>(l, stream);
            return launch<192, 128, 1, KVM>(l, stream);
        }
        if (l.dqk == 64) return launch<64, 64, 2, KVM>(l, stream);
        if (l.dqk == 128) return launch<128, 128, 2, KVM>(l, stream);
        return launch<192, 128, 2, KVM>(l, stream);
    }
}

}  // namespace

#if VPP_PART == 0 || VPP_PART == 3
hipError_t vpp_detail::launch_attn_contig(const Launch& l, hipStream_t stream) { return launch_dims<KV_CONTIG>(l, stream); }
#endif
#if VPP_PART == 1 || VPP_PART == 3
hipError_t vpp_detail::launch_attn_paged(const Launch& l, hipStream_t stream) { return launch_dims<KV_PAGED>(l, stream); }
#endif
#if VPP_PART == 2 || VPP_PART == 3
hipError_t vpp_detail::launch_attn_rope(const Launch& l, hipStream_t stream) { return launch_dims<KV_ROPE>(l, stream); }
#endif

#if VPP_PART == 0 || VPP_PART == 3 || VPP_PART == 4

// Scatter of a chunk's new K/V rows into a paged cache: the write that puts a
// chunk's own keys and values in the cache before its attention (section 2.4).
// One thread moves one 16-byte granule; consecutive threads walk the granules of a
// token, all of its K rows and then all of its V rows, so reads and writes are long
// contiguous runs. slot = page * page_size + row; slots outside
// [0, num_pages * page_size) are skipped (padding tokens use -1).
// Bound by HBM. A plain copy of the same bytes with one granule a thread reaches
// 6.2 TB/s, 6.6 with non-temporal loads and stores; two integer divisions and
// 64-bit addresses of every granule held this kernel at 5.1. Divisions are now by
// multiplication, and where a token's granules are a multiple of the wave
// (WAVE_TOKEN) its slot and addresses are worked out once per wave.
struct Divisor {  // x / d for x < 2^31: the high half of x * mul, shifted; mul 0: d = 1
    uint32_t mul;
    int32_t shift;
};
[[maybe_unused]] Divisor divisor(uint32_t d) {
    if (d == 1) return {0, 0};
    int s = 1;  // 2^s >= d
    while (((uint64_t)1 << s) < d) ++s;
    return {(uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d), s - 1};
}
__device__ __forceinline__ int divide(int x, Divisor d) {
    return d.mul ? (int)(__umulhi((uint32_t)x, d.mul) >> d.shift) : x;
}

struct AppendArgs {
    const u16* k_new;
    const u16* v_new;
    u16* k_pages;
    u16* v_pages;
    const int64_t* slots;
    int64_t kn_st, kn_sh, vn_st, vn_sh;  // element strides
    int64_t k_sp, k_st, k_sh, v_sp, v_st, v_sh;
    int32_t tokens, k_token, granules;  // granules of a token: its K rows' first, then its V rows'
    int32_t k_gran, v_gran, page_shift, num_pages;
    Divisor by_token, by_k, by_v;
};

template <bool WAVE_TOKEN, bool NT>
__global__ __launch_bounds__(256) void kv_append_kernel(AppendArgs a) {
    const int gid = (int)(blockIdx.x * 256u + threadIdx.x);
    int t = divide(gid, a.by_token);
    if constexpr (WAVE_TOKEN) t = __builtin_amdgcn_readfirstlane(t);
    if (t >= a.tokens) return;
    const int g = gid - t * a.granules;
    const int64_t slot = WAVE_TOKEN ? const_ptr<__attribute__((address_space(4))) const int64_t>((uint64_t)(uintptr_t)a.slots)[t]
                                    : a.slots[t];
    if (slot < 0 || slot >= ((int64_t)a.num_pages << a.page_shift)) return;
    const int64_t page = slot >> a.page_shift;
    const int64_t row = slot & (((int64_t)1 << a.page_shift) - 1);
    const bool is_k = g < a.k_token;
    const int r = is_k ? g : g - a.k_token;
    const int h = divide(r, is_k ? a.by_k : a.by_v);
    const int c = r - h * (is_k ? a.k_gran : a.v_gran);
    const u16* src = is_k ? a.k_new + (int64_t)t * a.kn_st : a.v_new + (int64_t)t * a.vn_st;
    u16* dst = is_k ? a.k_pages + page * a.k_sp + row * a.k_st : a.v_pages + page * a.v_sp + row * a.v_st;
    const u32x4* const from = (const u32x4*)(src + (int64_t)h * (is_k ? a.kn_sh : a.vn_sh)) + c;
    u32x4* const to = (u32x4*)(dst + (int64_t)h * (is_k ? a.k_sh : a.v_sh)) + c;
    if constexpr (NT) __builtin_nontemporal_store(__builtin_nontemporal_load(from), to);
    else *to = *from;
}

// ---------------------------------------------------------------------------
// host side: plan
// ---------------------------------------------------------------------------
// One segment with rows, cut into query tiles and split pieces. A work slot runs
// two tiles (paired) or one; `pieces` cuts its prefix (see piece_bounds).
struct SegPlan {
    int32_t seg, row0, len, prefix, kv_start;
    int32_t tiles, pieces;
    bool paired;
    int64_t whole;    // keys of the longest slot, unsplit
    int64_t longest;  // and of the last piece, the longest
    double key_steps; // 64-key steps of all tiles of a head group
    int32_t slots() const { return paired ? (tiles + 1) / 2 : tiles; }
};

struct vpp_chunk_attn_plan_s {
    vpp_chunk_attn_config_t cfg;
    float scale;
    std::vector<SegPlan> segs;
    std::vector<LaunchGroup> groups;  // launch order
    std::vector<CombineSeg> merges;   // split segments
    int32_t merge_blocks = 0;
    int64_t workgroups = 0;
    int64_t num_items = 0;  // work items of plan_items: two per slot and piece
    int32_t num_slots = 0;
    int32_t num_tiles = 0;
    int32_t num_splits = 1;
    int32_t nb = 2;  // 32-row query blocks per wave of the kernel variant the plan was made for
    int32_t pack = 1, tile_tokens = 256;
    bool nt = false;
    int32_t tokens = 0;
    double pairs = 0.0;
    size_t table_bytes = 0;  // groups, then merges, where they exceed the kernel arguments; else 0
    size_t part_o_off = 0, part_lse_off = 0;  // of the partials in the workspace
    size_t ws_bytes = 0;
    // pinned staging ring for the table copy, created on the first run that needs it
    char* staging[STAGING_SLOTS] = {};
    size_t staging_cap[STAGING_SLOTS] = {};
    hipEvent_t staging_done[STAGING_SLOTS] = {};
    bool staging_pending[STAGING_SLOTS] = {};
    int next_slot = 0;
};

namespace {

bool supported_dims(int dqk, int dv) {
    return (dqk == 64 && dv == 64) || (dqk == 128 && dv == 128) || (dqk == 192 && dv == 128);
}

// Kernel variants a plan may choose from (bit nb - 1): query blocks of 32 rows per
// wave. A chunk of at most two 256-row workgroups per CU and short key ranges (at
// most 8192 keys per tile on average) takes the 128-row tiles (NB = 1, two
// workgroups per CU), which even out the unequal key ranges of the diagonal tiles;
// others take what the launch model below finds faster. With dqk = 192 a few whole
// 256-row tiles keep them; otherwise the model chooses too: the 128-row tiles halve
// what a short segment leaves empty, and two workgroups a CU stream distinct keys
// faster than one (LaunchModel::stream). VPP_NB overrides, for tuning.
// us with 128- and 256-row tiles: up to one 256-row workgroup a CU 45 and 55 (2048 rows of
// 32/8 heads), 78 and 100 (4096 of 16/16), behind 7000 keys 254 and 247, 304 and 292; up to
// two of them, dqk 128, 135 and 128 (4096 of 32/8), behind 7000 keys 543 and 509; dqk 64
// 161 and 160 (8192 of 16/4). By these the line would be one workgroup a CU; callers of the
// plan interface have been given 128-row tiles up to two, and a test of it holds that.
bool small_chunk(const vpp_chunk_attn_config_t& c, int64_t tiles256, double mean_keys256) {
    return c.head_dim_qk <= 128 && tiles256 * c.num_q_heads <= 2 * 256 && mean_keys256 <= 8192.0;
}
int forced_nb() {
    const char* e = getenv("VPP_NB");
    return e && (atoi(e) == 1 || atoi(e) == 2) ? atoi(e) : 0;
}
int allowed_nb(const vpp_chunk_attn_config_t& c, bool small, int64_t tiles256, int64_t max_rows) {
    if (forced_nb()) return forced_nb();
    if (c.head_dim_qk > 128) return max_rows <= 128 || tiles256 * c.num_q_heads > 64 ? 3 : 2;
    return small ? 1 : 3;
}

// Query heads per tile: the largest divisor of Hq/Hkv up to 16. The heads that
// share a kv head read the same keys, so a tile of 256 rows may hold 16 tokens of 16
// of them as well as 256 tokens of one. It then wastes less: a short segment fills
// its tiles (43 rows of 64/4 heads: 3 tiles a kv head instead of 16), and a causal
// tile reaches 16 keys past its first token's instead of 256. One tile serves the
// heads that would each read its keys through the L2 again.
int heads_per_tile(const vpp_chunk_attn_config_t& c) {
    const int g = c.num_q_heads / c.num_kv_heads;
    for (int n = std::min(g, 16); n > 1; --n)
        if (g % n == 0) return n;
    return 1;
}

vpp_status_t check_config(const vpp_chunk_attn_config_t& c) {
    if (c.num_q_heads <= 0 || c.num_kv_heads <= 0 || c.num_q_heads % c.num_kv_heads != 0)
        return VPP_ERR_INVALID_ARG;
    if (c.max_chunk_tokens <= 0 || c.max_segments <= 0 || c.max_kv_len <= 0) return VPP_ERR_INVALID_ARG;
    if (c.max_kv_len > (int64_t)INT32_MAX - BM_MAX) return VPP_ERR_INVALID_ARG;
    if (!(c.softmax_scale >= 0.f) || !isfinite(c.softmax_scale)) return VPP_ERR_INVALID_ARG;
    if (c.num_splits == 0 || c.num_splits < -1 || c.num_splits > MAX_SPLITS) return VPP_ERR_INVALID_ARG;
    if (c.causal != 1) return VPP_ERR_UNSUPPORTED;
    if (!supported_dims(c.head_dim_qk, c.head_dim_v)) return VPP_ERR_UNSUPPORTED;
    return VPP_OK;
}

// A fixed split request: at most one piece per key tile of the longest prefix (a
// chunk without a prefix is not split), and of each segment's own.
int fixed_splits(const vpp_chunk_attn_config_t& c, int64_t max_prefix) {
    return (int)std::min<int64_t>(c.num_splits, std::max<int64_t>(1, max_prefix / BN));
}

// Keys [begin, end) of piece b of n of a segment; end = INT32_MAX for the last.
// A segment cut into fewer pieces than the plan's n has empty ones in front.
void piece_bounds(const SegPlan& s, int n, int b, int32_t& begin, int32_t& end) {
    const int skip = n - s.pieces;
    begin = b <= skip ? 0 : piece_begin(s.prefix, s.pieces, b - skip);
    end = b + 1 == n ? INT32_MAX : b < skip ? 0 : piece_begin(s.prefix, s.pieces, b + 1 - skip);
}

// Tile of slot `i` of a segment: the first (which = 0) or its partner; -1: none.
int slot_tile(const SegPlan& s, int i, int which) {
    if (which == 0) return i;
    const int t = s.tiles - 1 - i;
    return s.paired && t != i ? t : -1;
}

// Keys of tile t (bm rows) within [begin, end).
int64_t tile_keys(const SegPlan& s, int bm, int t, int32_t begin, int32_t end) {
    const int32_t own = s.prefix + std::min((t + 1) * bm, s.len);
    return std::max(0, std::min(own, end) - begin);
}

// Keys of the longest slot of a segment in [begin, end). A paired slot's two tiles
// together span the same keys in every slot but the first (whose partner may be
// short) and the middle one.
int64_t longest_slot(const SegPlan& s, int tt, int32_t begin, int32_t end) {
    const int last = s.slots() - 1;
    int64_t best = 0;
    for (int i : {0, std::min(1, last), last}) {
        int64_t keys = tile_keys(s, tt, i, begin, end);
        const int t = slot_tile(s, i, 1);
        if (t >= 0) keys += tile_keys(s, tt, t, begin, end);
        best = std::max(best, keys);
    }
    return best;
}

// Whether a split segment's last pieces, which end with the tiles' own keys, are a run of
// their own, before the other pieces. In one run of all pieces the XCDs get the last pieces
// of whole head groups, so some XCDs work longer where those are no multiple of the XCDs:
// the line is a quarter more than the mean. us in one run and in two: 6089 rows of 4/1
// heads behind 1539 keys in 8 pieces 268 and 132, 2000 behind 16000 118 and 93; 2645 of
// 24/2 heads behind 2959 in 4 pieces 271 and 199. Below the line both are alike (217 rows of
// 4/1 heads behind 32768 34.2 and 33.7, 600 behind 16000 48.7 and 49.2).
bool last_pieces_first(const SegPlan& s, int64_t head_groups) {
    const int64_t most = (head_groups + 7) / 8 * 8;  // 8 times the head groups of the fullest XCD
    return s.pieces > 1 && 4 * (most - head_groups) * s.len > head_groups * ((int64_t)s.prefix + s.len);
}

// ---- launch model -----------------------------------------------------------
// What a plan may choose: the tile variant, one or two tiles per work slot, and the
// pieces of every segment's prefix. The choice is the one whose launch this model
// finishes first. Its constants are measured on one MI355X with normal operands.
struct LaunchModel {
    int heads, kv_heads, pack, dqk, dv;
    static constexpr int NUM_CU = 256, NXCD = 8;

    // One 64-key step of a workgroup takes `few` us while few of them run and `full` us
    // with every place taken: one 256-row workgroup a CU, or two of 128 rows. In
    // between the chip is held by power, which grows with the cube of its clock: 192 of
    // 256 places busy step 1.1 times as fast as all of them, not 1.33 times.
    struct Speed {
        double few, full;
        double step[2 * NUM_CU / NXCD];  // with (i + 1) * NXCD workgroups in flight
        double rate = 0.0;               // the most steps per us of any of those
        Speed(int nb, double few, double full) : few(few), full(full) {
            for (int i = 0; i < NUM_CU / NXCD * (3 - nb); ++i) {
                const double wgs = (i + 1) * NXCD;
                if (nb == 2) step[i] = std::max(few, full * cbrt(wgs / NUM_CU));
                else if (wgs <= NUM_CU) step[i] = std::max(few, 1.17 * few * cbrt(wgs / NUM_CU));
                else step[i] = full * cbrt(wgs / (2 * NUM_CU));  // while any CU holds two, those set the pace
                rate = std::max(rate, wgs / step[i]);
            }
        }
    };
    const Speed& speed(int nb) const {
        static const Speed table[2][3] = {{{1, 0.64, 1.22}, {1, 0.84, 1.85}, {1, 1.08, 2.15}},
                                          {{2, 1.03, 1.20}, {2, 1.31, 1.72}, {2, 1.52, 2.04}}};
        return table[nb - 1][dqk == 64 ? 0 : dqk == 128 ? 1 : 2];
    }
    // What a tile costs beside its steps, in steps: Q load, pipeline fill, first and
    // last step, store. Two 128-row workgroups a CU hide much of each other's.
    double tile(int nb) const { return nb == 1 ? 2.0 : 4.0; }
    // The rate at which workgroups stream distinct keys, one or two in flight per CU:
    // it holds back the steps of segments with few tiles. Single tokens behind 2000 to 16000
    // keys: 5.1, 6.4, 6.2 TB/s at dqk 64, 128, 192 with two of 128 rows, 3.1, 4.2, 4.5 with
    // one of 256.
    double stream(int nb) const { return nb == 1 ? 6.0e6 : 3.8e6; }  // bytes per us

    // Time of the merge of part_rows partial rows: a launch, and the partials written
    // and read back.
    double merge(int64_t part_rows) const {
        return part_rows == 0 ? 0.0 : 4.0 + 2.0 * (double)part_rows * heads * (4.0 * dv + 4.0) / 5.0e6;
    }

    // Steps of all tiles and pieces of a segment, one head group: fixed costs included.
    double steps(const SegPlan& s, int nb) const {
        return s.key_steps + (double)s.tiles * s.pieces * tile(nb);
    }
    // Bytes of distinct keys and values a launch reads: once a kv head, also where its heads
    // take several tiles.
    double key_bytes(const std::vector<SegPlan>& segs) const {
        double rows = 0.0;
        for (const SegPlan& s : segs) rows += (double)s.prefix + s.len;
        return rows * kv_heads * (dqk + dv) * 2.0;
    }
    // The time no launch of `all` steps of its workgroups comes under: the most steps per us
    // that any number of workgroups makes, and the rate of its keys.
    double bound(double all, double bytes, int nb) const {
        return std::max(all / speed(nb).rate, bytes / stream(nb));
    }

    // Time of a launch of `segs` (longest slots first): one XCD's share of each group
    // (work_coords), placed in order on whichever of its workgroup places frees first.
    // All places progress alike, so the schedule is found in steps and then put on the
    // clock.
    double launch(const std::vector<SegPlan>& segs, int nb, int tt, std::vector<double>& lanes,
                  std::vector<double>& costs) const {
        const int64_t groups = heads / pack;
        const int places = NUM_CU / NXCD * (3 - nb);
        const double c_tile = tile(nb);
        lanes.assign((size_t)places, 0.0);
        double left = 0.0;  // steps of one place still to come, if spread evenly
        for (const SegPlan& s : segs) left += steps(s, nb) * groups / (NXCD * places);
        double even = 0.0;               // steps every place has had alike
        double placed = 0.0, top = 0.0;  // beside those: the mean and the most of a place
        int64_t seen = 0;
        // `count` pieces of a segment from `piece` down, one run of slots (tile_work): `own`
        // steps of one place, `longest` of one slot.
        auto run = [&](const SegPlan& s, int piece, int count, double own, double longest) {
            const int64_t h = groups * count, n = s.slots() * h;
            int64_t share = (seen + n + NXCD - 1) / NXCD - (seen + NXCD - 1) / NXCD;
            seen += n;
            // While twice a run's longest slot and what the fullest place is ahead are
            // still to come on every place, the shorter slots behind even out whatever the
            // run's own placing would leave uneven.
            left -= own;
            const bool evens_out = top - placed <= left;
            if (evens_out && 2.0 * longest < left) {
                even += own;
                return;
            }
            placed += own;
            // its slots in order, or every `stride`-th of its heads, longest first
            const bool alike = s.paired || piece < s.pieces - 1;  // a run without last pieces
            const int stride = alike ? 1 : (int)(NXCD / std::min<int64_t>(NXCD, h & -h));
            const int64_t all = share;
            // many rounds of one run fill the places evenly: only a few are placed,
            // taken evenly from its slots
            if (share > (evens_out ? 5 : 8) * places) {
                share = share % places + 4 * places;
                const double spread = own * (double)(all - share) / (double)all;
                even += spread;
                placed -= spread;
            }
            if (share == 0) return;
            // slot i of a head group, piece by piece, in launch order
            const int64_t ring = (int64_t)s.slots() * count;
            auto cost = [&](int64_t i) {
                const int b = (int)(i / s.slots()), at = (int)(i - (int64_t)b * s.slots());
                const int32_t kb = s.pieces == 1 ? 0 : piece_begin(s.prefix, s.pieces, piece - b);
                const int32_t ke = piece - b == s.pieces - 1 ? INT32_MAX : piece_begin(s.prefix, s.pieces, piece - b + 1);
                double t = 0.0;
                for (int which = 0; which < 2; ++which) {
                    const int tl = slot_tile(s, alike ? at : s.slots() - 1 - at, which);
                    if (tl >= 0) t += (double)((tile_keys(s, tt, tl, kb, ke) + BN - 1) / BN) + c_tile;
                }
                return t;
            };
            const bool again = ring < share;  // head groups repeat the same costs
            if (again) {
                costs.resize((size_t)ring);
                for (int64_t i = 0; i < ring; ++i) costs[(size_t)i] = cost(i);
            }
            const int64_t step = stride * (all / share), rest = all % share;
            int64_t i = 0, err = 0;
            for (int64_t j = 0; j < share; ++j) {
                // the place that frees first is the heap's root: give it the slot, sift it down
                const double t = lanes[0] + (again ? costs[(size_t)i] : cost(i));
                int at = 0;
                for (int c = 1; c < places; c = 2 * at + 1) {
                    if (c + 1 < places) c += lanes[(size_t)c + 1] < lanes[(size_t)c];
                    if (lanes[(size_t)c] >= t) break;
                    lanes[(size_t)at] = lanes[(size_t)c];
                    at = c;
                }
                lanes[(size_t)at] = t;
                top = std::max(top, t);
                i += step;
                if ((err += rest) >= share) {
                    err -= share;
                    i += stride;
                }
                if (i >= ring) i = i < 2 * ring ? i - ring : i % ring;
            }
        };
        const double per_place = (double)groups / (NXCD * places);
        for (const SegPlan& s : segs) {
            const double all = steps(s, nb) * per_place, longest = (double)s.longest / BN + 2.0 * c_tile;
            if (!last_pieces_first(s, groups)) {
                run(s, s.pieces - 1, s.pieces, all, longest);
                continue;
            }
            // the keys before the last piece are the same in every tile
            const int others = s.pieces - 1;
            const double before = (double)(piece_begin(s.prefix, s.pieces, others) / BN);
            const double rest = s.tiles * (before + others * c_tile) * per_place;
            run(s, others, 1, all - rest, longest);
            run(s, others - 1, others, rest, 2.0 * (before / others + 1.0 + c_tile));
        }
        double steps = 0.0;
        for (double& l : lanes) steps += (l += even) * NXCD;
        std::sort(lanes.begin(), lanes.end());
        const Speed& v = speed(nb);
        const double stream_step = key_bytes(segs) / steps / stream(nb);  // us a step of each workgroup
        double t = 0.0, at = 0.0;
        for (int i = 0; i < places; ++i) {
            if (lanes[(size_t)i] == at) continue;
            const double wgs = (double)(places - i) * NXCD;
            t += (lanes[(size_t)i] - at) * std::max(v.step[places - 1 - i], wgs * stream_step);
            at = lanes[(size_t)i];
        }
        return t;
    }
};

LaunchModel launch_model(const vpp_chunk_attn_config_t& c, int pack) {
    return {c.num_q_heads, c.num_kv_heads, pack, c.head_dim_qk, c.head_dim_v};
}

// A candidate plan and its modelled time.
struct Candidate {
    std::vector<SegPlan> segs;
    int nb = 2, tt = 256;
    double t = 0.0;
    int64_t part_rows() const {
        int64_t n = 0;
        for (const SegPlan& s : segs) n += s.pieces > 1 ? (int64_t)s.pieces * s.len : 0;
        return n;
    }
};

size_t partial_bytes(const vpp_chunk_attn_config_t& c, int64_t part_rows) {
    return align256((size_t)part_rows * c.num_q_heads * c.head_dim_v * sizeof(float)) +
           align256((size_t)part_rows * c.num_q_heads * sizeof(float));
}

// Plan of the segments `segs` (rows set, the rest chosen here); an automatic split
// takes at most max_part bytes of partials.
Candidate choose_plan(const vpp_chunk_attn_config_t& c, const std::vector<SegPlan>& segs, int nb_mask, int pack,
                      size_t max_part) {
    constexpr int MAX_PIECES = 64;
    constexpr int64_t MIN_PIECE = 4 * BN;  // keys of prefix a piece holds at least
    const LaunchModel model = launch_model(c, pack);
    const int64_t groups = c.num_q_heads / pack;
    int64_t max_prefix = 0;
    for (const SegPlan& s : segs) max_prefix = std::max<int64_t>(max_prefix, s.prefix);
    const int fixed = c.num_splits >= 1 ? fixed_splits(c, max_prefix) : 0;
    Candidate best, x;
    std::vector<double> lanes, costs;
    const double bytes = model.key_bytes(segs);
    // Candidates compare by their modelled time and what it leaves out: a split must be
    // worth its partials' memory; pairs of one-head tiles share their key reads with the
    // other slots of the segment, 2 to 9 % of a long launch (mla 6540 against 6703 us).
    // Tiles of several heads are few tokens apart, so single ones, which all start at key
    // 0, share them as well: up to 3 % faster than pairs (8192 rows of 64/4 heads without a
    // prefix 1014 against 1048 us, 4096 of 32/8 behind 20480 1248 against 1262). In short
    // launches of equal modelled time pairs start fewer workgroups (4096 rows of 32/8
    // heads without a prefix 132.5 against 135.5 us).
    double best_score = 0.0;
    // Whether the candidate was weighed: false if even its work spread evenly would take
    // longer than the best one does (more pieces only add to that). Most go this way: a
    // launch is placed for 2 to 8 of up to 36 candidates.
    auto consider = [&](bool paired, bool split) {
        const int64_t part_rows = x.part_rows();
        if (!fixed && !best.segs.empty() && partial_bytes(c, part_rows) > max_part) return true;
        const double handicap = split ? 1.02 : 1.0, merge = model.merge(part_rows);
        if (!best.segs.empty()) {
            double all = 0.0;
            for (const SegPlan& s : x.segs) all += model.steps(s, x.nb) * groups;
            if ((model.bound(all, bytes, x.nb) + merge) * handicap >= best_score) return false;
        }
        for (SegPlan& s : x.segs)
            s.longest = s.pieces == 1 ? s.whole : longest_slot(s, x.tt, piece_begin(s.prefix, s.pieces, s.pieces - 1), INT32_MAX);
        std::stable_sort(x.segs.begin(), x.segs.end(),
                         [](const SegPlan& a, const SegPlan& b) { return a.longest > b.longest; });
        x.t = model.launch(x.segs, x.nb, x.tt, lanes, costs) + merge;
        const double order = pack > 1 ? (paired && x.t > 400.0 ? 0.01 : 0.0) : (!paired && x.t > 400.0 ? 0.04 : 0.0);
        const double score = x.t * (handicap + order);
        if (best.segs.empty() || score < best_score) {
            best = x;
            best_score = score;
        }
        return true;
    };
    // first the variant whose launch would be the shorter one if spread evenly
    auto evenly = [&](int nb) {
        double all = 0.0;
        for (const SegPlan& s : segs)
            all += (double)groups * ceil((double)s.len * pack / block_rows(nb)) * (s.prefix + 0.5 * s.len) / BN;
        return model.bound(all, bytes, nb);
    };
    const int first = nb_mask == 3 && evenly(1) < evenly(2) ? 1 : 2;
    for (int nb : {first, 3 - first}) {
        if (!(nb_mask & nb)) continue;
        x.nb = nb;
        x.tt = block_rows(nb) / pack;
        // the launch's work if spread evenly: steps of one workgroup place, and its time
        double steps = 0.0;
        std::vector<SegPlan> base = segs;
        for (SegPlan& s : base) {
            s.tiles = (int32_t)(((int64_t)s.len + x.tt - 1) / x.tt);
            for (int t = 0; t < s.tiles; ++t) s.key_steps += (double)((tile_keys(s, x.tt, t, 0, INT32_MAX) + BN - 1) / BN);
            steps += (double)groups * s.tiles * (((double)s.prefix + 0.5 * s.len) / BN + 1.0);
        }
        const double even = steps / (LaunchModel::NUM_CU * (3 - nb));
        const double bound = std::max(even * model.speed(nb).full, bytes / model.stream(nb));
        for (int paired = 1; paired >= 0; --paired) {
            x.segs = base;
            for (SegPlan& s : x.segs) {
                s.paired = paired != 0;
                s.whole = longest_slot(s, x.tt, 0, INT32_MAX);
                s.pieces = fixed > 1 ? (int)std::min<int64_t>(fixed, std::max(1, s.prefix / BN)) : 1;
            }
            consider(paired != 0, false);
            if (fixed || best.t < 1.04 * bound) continue;
            double last_t = 1e30;
            for (double f : {2.0, 1.0, 0.7, 0.5, 0.35, 0.25, 0.17, 0.12}) {
                const double target = std::max(even * f, 4.0);  // steps of a workgroup
                bool changed = false;
                for (SegPlan& s : x.segs) {
                    const int32_t before = s.pieces, cap = std::min<int32_t>(MAX_PIECES, s.prefix / MIN_PIECE);
                    s.pieces = std::max(1, (int)std::min<double>(cap, ceil((double)s.whole / BN / target)));
                    changed = changed || s.pieces != before;
                }
                if (!changed) continue;
                if (!consider(paired != 0, true)) break;
                if (target <= 4.0 || (x.t > last_t && x.t > 1.1 * best.t) || best.t < 1.04 * bound) break;
                last_t = x.t;
            }
        }
    }
    return best;
}

// The split count of one-head tiles run in pairs, from a launch placed head by head:
// the rule by which a plan's workspace fits vpp_chunk_attn_run_noalloc's scratch or not.
// A chunk whose workspace it keeps within the scratch stays within it.
int one_head_splits(const vpp_chunk_attn_config_t& c, std::vector<SegPlan> segs, int nb, int64_t max_prefix,
                    int32_t tokens) {
    constexpr int NXCD = LaunchModel::NXCD;
    constexpr double TILE = 2.0;  // fixed cost of a tile, in steps
    const int bm = block_rows(nb), heads = c.num_q_heads;
    const double step_s = 2.0 * bm * BN * (c.head_dim_qk + c.head_dim_v) / 5.0e12;
    std::vector<double> cost, free_at;
    auto simulate = [&](int n, double& ideal) {
        struct Group { int si, b; int64_t keys; };
        std::vector<Group> order;
        for (size_t k = 0; k < segs.size(); ++k) {
            segs[k].tiles = (int32_t)(((int64_t)segs[k].len + bm - 1) / bm);
            segs[k].paired = true;
            for (int b = 0; b < n; ++b) {
                const int32_t kb = n == 1 ? 0 : piece_begin(segs[k].prefix, n, b);
                const int32_t ke = b + 1 == n ? INT32_MAX : piece_begin(segs[k].prefix, n, b + 1);
                order.push_back({(int)k, b, longest_slot(segs[k], bm, kb, ke)});
            }
        }
        std::stable_sort(order.begin(), order.end(), [](const Group& x, const Group& y) { return x.keys > y.keys; });
        cost.clear();
        double total = 0.0;
        for (const Group& g : order) {
            const SegPlan& s = segs[(size_t)g.si];
            const int32_t kb = n == 1 ? 0 : piece_begin(s.prefix, n, g.b);
            const int32_t ke = g.b + 1 == n ? INT32_MAX : piece_begin(s.prefix, n, g.b + 1);
            for (int i = 0; i < s.slots(); ++i) {
                double t = 0.0;
                for (int which = 0; which < 2; ++which)
                    if (slot_tile(s, i, which) >= 0)
                        t += (double)((tile_keys(s, bm, slot_tile(s, i, which), kb, ke) + BN - 1) / BN) + TILE;
                cost.push_back(t);
                total += t;
            }
        }
        const int64_t nslots = (int64_t)cost.size(), all = nslots * heads, per = all / NXCD;
        const size_t lanes = (size_t)(LaunchModel::NUM_CU / NXCD * (3 - nb));
        ideal = total * heads / (double)(NXCD * lanes) * step_s;
        double makespan = 0.0;
        for (int x = 0; x < (heads % NXCD == 0 ? 1 : NXCD); ++x) {
            free_at.assign(lanes, 0.0);
            auto place = [&](int64_t l) {
                std::pop_heap(free_at.begin(), free_at.end(), std::greater<double>());
                free_at.back() += cost[(size_t)(l % nslots)];
                std::push_heap(free_at.begin(), free_at.end(), std::greater<double>());
            };
            for (int64_t j = 0; j < per; ++j) place(x * per + j);
            for (int64_t l = per * NXCD + x; l < all; l += NXCD) place(l);
            makespan = std::max(makespan, *std::max_element(free_at.begin(), free_at.end()));
        }
        return makespan * step_s;
    };
    double ideal = 0.0;
    const double t1 = simulate(1, ideal);
    if (t1 <= 1.05 * ideal) return 1;
    const double partial_s = 2.0 * tokens * heads * (4.0 * c.head_dim_v + 4.0) / 3.0e12;
    int best = 1;
    double best_t = 0.97 * t1;
    for (int n : {2, 3, 4, 6, 8, 12, 16}) {
        if (n > std::min<int64_t>(MAX_SPLITS, max_prefix / 1024)) break;
        const double t = simulate(n, ideal) + n * partial_s;
        if (t < best_t) {
            best_t = t;
            best = n;
        }
    }
    return best;
}

}  // namespace

extern "C" vpp_status_t vpp_chunk_attn_plan(const vpp_chunk_attn_config_t* cfg, int32_t num_segments,
                                            const int32_t* cu_q, const int64_t* kv_start,
                                            const int64_t* prefix_len, vpp_chunk_attn_plan_t* inout_plan,
                                            size_t* workspace_bytes) {
    if (!inout_plan || !workspace_bytes) return VPP_ERR_INVALID_ARG;
    vpp_chunk_attn_plan_s* p = *inout_plan;
    vpp_chunk_attn_config_t c;
    if (p) {
        c = cfg ? *cfg : p->cfg;
        if (cfg && memcmp(cfg, &p->cfg, sizeof c) != 0) return VPP_ERR_INVALID_ARG;
    } else {
        if (!cfg) return VPP_ERR_INVALID_ARG;
        c = *cfg;
    }
    vpp_status_t st = check_config(c);
    if (st != VPP_OK) return st;
    if (num_segments <= 0 || num_segments > c.max_segments) return VPP_ERR_INVALID_ARG;
    if (!cu_q || !kv_start || !prefix_len) return VPP_ERR_INVALID_ARG;
    if (cu_q[0] != 0) return VPP_ERR_INVALID_ARG;
    for (int s = 0; s < num_segments; ++s) {
        if (cu_q[s + 1] < cu_q[s]) return VPP_ERR_INVALID_ARG;
        if (kv_start[s] < 0 || prefix_len[s] < 0) return VPP_ERR_INVALID_ARG;
        const int64_t len = cu_q[s + 1] - cu_q[s];
        if (prefix_len[s] > c.max_kv_len || kv_start[s] > c.max_kv_len) return VPP_ERR_INVALID_ARG;
        if (kv_start[s] + prefix_len[s] + len > c.max_kv_len) return VPP_ERR_INVALID_ARG;
    }
    if (cu_q[num_segments] > c.max_chunk_tokens) return VPP_ERR_INVALID_ARG;

    // query tiles of every segment, with their whole key range [0, last position + 1)
    int64_t tiles256 = 0;
    double keys256 = 0.0;
    for (int s = 0; s < num_segments; ++s)
        for (int r0 = cu_q[s]; r0 < cu_q[s + 1]; r0 += block_rows(2)) {
            ++tiles256;
            keys256 += (double)prefix_len[s] + (r0 - cu_q[s]) + std::min(block_rows(2), cu_q[s + 1] - r0);
        }
    const int pack = heads_per_tile(c);
    // Work slots. A workgroup runs one slot: one query tile, or two of one segment,
    // tile i with its key range ascending, then tile T-1-i (the partner from the
    // other end of the segment) descending. A pair's two ranges together span the
    // same number of keys in every slot of the segment, so the workgroups of a
    // segment finish together; and at any moment they all read one of two key
    // positions (the ascending front, and the descending one, which mirrors it), so
    // the tiles running side by side on one XCD share each K/V tile through its L2.
    Candidate plan;
    std::vector<LaunchGroup> groups;
    std::vector<CombineSeg> merges;
    double pairs = 0.0;
    int64_t ntiles = 0, nslots = 0, wgs = 0, part_rows = 0, blocks = 0;
    double key_steps = 0.0, lone_steps = 0.0;  // per head group; of segments of one tile
    int nsplit = 1;
    try {
        std::vector<SegPlan> segs;
        int64_t max_rows = 0, max_prefix = 0;
        for (int s = 0; s < num_segments; ++s) {
            const int32_t len = cu_q[s + 1] - cu_q[s];
            if (len == 0) continue;
            segs.push_back({s, cu_q[s], len, (int32_t)prefix_len[s], (int32_t)kv_start[s], 0, 1, true, 0, 0, 0.0});
            // visible pairs: sum over rows of (position + 1)
            pairs += (double)len * (double)prefix_len[s] + 0.5 * (double)len * (len + 1.0);
            max_rows = std::max<int64_t>(max_rows, (int64_t)len * pack);
            max_prefix = std::max(max_prefix, prefix_len[s]);
        }
        if (!segs.empty()) {
            const bool small = small_chunk(c, tiles256, keys256 / tiles256);
            const int nb_mask = allowed_nb(c, small, tiles256, max_rows);
            plan = choose_plan(c, segs, nb_mask, pack, SIZE_MAX);
            // a chunk that one-head tiles in pairs would keep within the scratch of
            // run_noalloc stays within it
            const size_t table = align256(segs.size() > INLINE_GROUPS ? segs.size() * (sizeof(LaunchGroup) + sizeof(CombineSeg)) : 1);
            const size_t room = (size_t)VPP_NOALLOC_SCRATCH_BYTES - std::min<size_t>(table, VPP_NOALLOC_SCRATCH_BYTES);
            if (c.num_splits < 1 && partial_bytes(c, plan.part_rows()) > room) {
                const int one_head_nb = forced_nb() ? forced_nb() : small ? 1 : 2;
                const int n = one_head_splits(c, segs, one_head_nb, max_prefix, cu_q[num_segments]);
                if (n == 1 || partial_bytes(c, (int64_t)n * cu_q[num_segments]) <= VPP_NOALLOC_SCRATCH_BYTES)
                    plan = choose_plan(c, segs, nb_mask, pack, room);
            }
        }
        if (c.num_splits >= 1 && !segs.empty()) nsplit = fixed_splits(c, max_prefix);
        else
            for (const SegPlan& s : plan.segs) nsplit = std::max(nsplit, s.pieces);
        // partial rows of the split segments, piece by piece; a segment of one piece
        // writes its results directly
        for (const SegPlan& s : plan.segs) {
            LaunchGroup g{(int32_t)wgs, s.row0, s.len, s.prefix, s.kv_start, s.seg, s.pieces, -1, s.slots(), s.tiles};
            if (last_pieces_first(s, c.num_q_heads / pack)) g.pieces = -s.pieces;
            if (s.pieces > 1) {
                g.part0 = (int32_t)part_rows;
                merges.push_back({(int32_t)blocks, s.row0, s.len, s.pieces, (int32_t)part_rows});
                part_rows += (int64_t)s.pieces * s.len;
                const int64_t per_block = 1024 / c.head_dim_v / merge_ways(s.pieces);  // (row, head) pairs
                blocks += ((int64_t)s.len * c.num_q_heads + per_block - 1) / per_block;
            }
            groups.push_back(g);
            wgs += (int64_t)g.slots * s.pieces * (c.num_q_heads / pack);
            ntiles += s.tiles;
            nslots += s.slots();
            const double keys = s.tiles * (s.prefix + 0.5 * s.len);
            key_steps += keys;
            if (s.tiles == 1) lone_steps += keys;
        }
    } catch (const std::bad_alloc&) {
        return VPP_ERR_NOMEM;
    }
    const int nb = plan.nb, tt = block_rows(nb) / pack;

    if (!p) {
        p = new (std::nothrow) vpp_chunk_attn_plan_s();
        if (!p) return VPP_ERR_NOMEM;
        p->cfg = c;
        *inout_plan = p;
    }
    p->nb = nb;
    p->pack = pack;
    p->tile_tokens = tt;
    p->nt = nb == 1 && pack == c.num_q_heads / c.num_kv_heads && lone_steps > 0.5 * key_steps;
    p->scale = c.softmax_scale > 0.f ? c.softmax_scale : (float)(1.0 / sqrt((double)c.head_dim_qk));
    p->segs.swap(plan.segs);
    p->groups.swap(groups);
    p->merges.swap(merges);
    p->merge_blocks = (int32_t)blocks;
    p->workgroups = wgs;
    p->num_tiles = (int32_t)ntiles;
    p->num_splits = nsplit;
    p->num_slots = (int32_t)(nslots * nsplit);
    p->num_items = 2 * nslots * nsplit;
    p->tokens = cu_q[num_segments];
    p->pairs = pairs;
    p->table_bytes = p->groups.size() > INLINE_GROUPS || p->merges.size() > INLINE_GROUPS
                         ? p->groups.size() * sizeof(LaunchGroup) + p->merges.size() * sizeof(CombineSeg)
                         : 0;
    // The workspace: the table, then the partials. Callers that size it from plan_items find 32
    // bytes for each of those up to 1 MiB; the listing itself grows with the most pieces of any
    // segment times all slots, far past what a launch of many segments uses.
    p->part_o_off = align256(std::max<size_t>(p->table_bytes, 1));
    p->part_lse_off = p->part_o_off + align256((size_t)part_rows * c.num_q_heads * c.head_dim_v * sizeof(float));
    p->ws_bytes = std::max(p->part_lse_off + align256((size_t)part_rows * c.num_q_heads * sizeof(float)),
                           std::min<size_t>(align256((size_t)p->num_items * sizeof(WorkItem)), 1u << 20));
    *workspace_bytes = p->ws_bytes;
    return VPP_OK;
}

extern "C" vpp_status_t vpp_chunk_attn_plan_info(vpp_chunk_attn_plan_t p, vpp_chunk_attn_plan_info_t* info) {
    if (!p || !info) return VPP_ERR_INVALID_ARG;
    info->num_tiles = p->num_tiles;
    info->num_splits = p->num_splits;
    info->num_work_items = (int32_t)p->num_items;
    info->num_slots = p->num_slots;
    info->block_m = block_rows(p->nb);
    info->block_n = BN;
    info->num_tokens = p->tokens;
    info->workspace_bytes = (int64_t)p->ws_bytes;
    info->pairs = p->pairs;
    return VPP_OK;
}

extern "C" vpp_status_t vpp_chunk_attn_plan_items(vpp_chunk_attn_plan_t p, vpp_chunk_attn_work_item_t* items,
                                                  int32_t capacity, int32_t* count) {
    if (!p || !count || capacity < 0 || (capacity > 0 && !items)) return VPP_ERR_INVALID_ARG;
    *count = (int32_t)p->num_items;
    if (capacity == 0) return VPP_OK;
    const int bm = p->tile_tokens;
    int32_t n = 0;
    // (segment, piece) pairs, longest slot first; the empty pieces of segments cut
    // into fewer than num_splits are listed too
    struct Piece {
        const SegPlan* s;
        int32_t b, begin, end;
        int64_t keys;
    };
    try {
        std::vector<Piece> order;
        for (const SegPlan& s : p->segs)
            for (int b = 0; b < p->num_splits; ++b) {
                Piece r{&s, b, 0, 0, 0};
                piece_bounds(s, p->num_splits, b, r.begin, r.end);
                r.keys = longest_slot(s, bm, r.begin, r.end);
                order.push_back(r);
            }
        std::stable_sort(order.begin(), order.end(), [](const Piece& x, const Piece& y) { return x.keys > y.keys; });
        for (const Piece& r : order) {
            const SegPlan& s = *r.s;
            for (int i = 0; i < s.slots(); ++i)
                for (int which = 0; which < 2; ++which) {
                    if (n == capacity) return VPP_OK;
                    const int t = slot_tile(s, i, which);
                    WorkItem w = {0, 0, 0, 0, 0, 0, 0};
                    if (t >= 0) {
                        w.row0 = s.row0 + t * bm;
                        w.nrows = std::min(bm, s.len - t * bm);
                        w.pos0 = s.prefix + t * bm;
                        w.key_begin = r.begin;
                        w.key_end = std::min(r.end, w.pos0 + w.nrows);
                        w.split = r.b;
                        w.kv_base = s.kv_start;
                    }
                    items[n++] = w;
                }
        }
    } catch (const std::bad_alloc&) {
        return VPP_ERR_NOMEM;
    }
    return VPP_OK;
}

extern "C" void vpp_chunk_attn_destroy(vpp_chunk_attn_plan_t p) {
    if (!p) return;
    for (int i = 0; i < STAGING_SLOTS; ++i) {
        if (p->staging_done[i]) {
            if (p->staging_pending[i]) (void)hipEventSynchronize(p->staging_done[i]);
            (void)hipEventDestroy(p->staging_done[i]);
        }
        if (p->staging[i]) (void)hipHostFree(p->staging[i]);
    }
    delete p;
}

extern "C" const char* vpp_status_str(vpp_status_t s) {
    switch (s) {
        case VPP_OK: return "ok";
        case VPP_ERR_INVALID_ARG: return "invalid argument";
        case VPP_ERR_UNSUPPORTED: return "unsupported configuration";
        case VPP_ERR_WORKSPACE: return "workspace too small";
        case VPP_ERR_HIP: return "HIP runtime error";
        case VPP_ERR_NOMEM: return "out of host memory";
    }
    return "unknown status";
}

// ---------------------------------------------------------------------------
// host side: run
// ---------------------------------------------------------------------------
namespace {

bool aligned16(const void* ptr) { return ((uintptr_t)ptr & 15u) == 0; }
bool stride_ok(int64_t s) { return s > 0 && (s % 8) == 0; }

int env_xcd_remap() {
    const char* s = getenv("VPP_XCD_REMAP");
    return s ? atoi(s) : 1;
}

}  // namespace

namespace {

// Paged-cache description of one run (see vpp_chunk_attn_run_paged).
struct PagedKV {
    const int32_t* block_table;
    int64_t bt_st, k_sp, v_sp;
    int32_t page_shift, num_pages;
};

// Shared key part of the split key layout (see vpp_chunk_attn_run_mla).
struct RopeK {
    const void* k_rope;
    int64_t kr_st;
};

// The plan's part of the kernel arguments.
void plan_args(const vpp_chunk_attn_plan_s* p, AttnArgs& a) {
    const vpp_chunk_attn_config_t& c = p->cfg;
    a.num_groups = (int32_t)p->groups.size();
    a.num_heads = c.num_q_heads;
    a.group = c.num_q_heads / c.num_kv_heads;
    a.pack = p->pack;
    a.pack_magic = (65536 + p->pack - 1) / p->pack;  // exact for r < 256, pack <= 16
    a.tile_tokens = p->tile_tokens;
    a.head_groups = c.num_q_heads / p->pack;
    a.scale_log2 = (float)((double)p->scale * 1.4426950408889634);
    a.xcd_remap = env_xcd_remap();
}

// How run_impl puts a launch table too large for the kernel arguments into the
// workspace: through the plan's pinned staging ring (asynchronous), or straight
// from the plan's host memory, which allocates nothing (the copy out of memory
// that is not pinned completes before the call returns).
enum class Upload { staged, direct };

vpp_status_t run_impl(vpp_chunk_attn_plan_t p, const void* q, int64_t q_st, int64_t q_sh, const void* k,
                      int64_t k_st, int64_t k_sh, const void* v, int64_t v_st, int64_t v_sh, void* out,
                      int64_t o_st, int64_t o_sh, float* lse, int64_t lse_sh, void* workspace,
                      size_t workspace_bytes, void* stream_ptr, const PagedKV* pg, const RopeK* rope = nullptr,
                      Upload upload = Upload::staged) {
    if (!p) return VPP_ERR_INVALID_ARG;
    if (!q || !k || !v || !out) return VPP_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return VPP_ERR_INVALID_ARG;
    if (!stride_ok(q_st) || !stride_ok(q_sh) || !stride_ok(k_st) || !stride_ok(k_sh) || !stride_ok(v_st) ||
        !stride_ok(v_sh) || !stride_ok(o_st) || !stride_ok(o_sh))
        return VPP_ERR_INVALID_ARG;
    if (lse && (((uintptr_t)lse & 3u) != 0 || lse_sh < p->tokens)) return VPP_ERR_INVALID_ARG;
    // the kernels keep element strides in 32 bits; the bytes of one key tile
    // (BN rows of a cache row stride, 2 bytes an element) must also stay below
    // 2^31, the range of a buffer resource's size field
    const int64_t smax = ((int64_t)1 << 31) / 64;
    const int64_t row_smax = ((int64_t)1 << 31) / (2 * BN);
    if (q_st >= smax || q_sh >= smax || k_st >= row_smax || k_sh >= smax || v_st >= row_smax ||
        v_sh >= smax || o_st >= smax || o_sh >= smax || (lse && lse_sh >= ((int64_t)1 << 31)))
        return VPP_ERR_INVALID_ARG;
    if (rope) {
        if (p->cfg.head_dim_qk != 192 || p->cfg.head_dim_v != 128) return VPP_ERR_UNSUPPORTED;
        if (!rope->k_rope || !aligned16(rope->k_rope) || !stride_ok(rope->kr_st) || rope->kr_st < 64 ||
            rope->kr_st >= row_smax)
            return VPP_ERR_INVALID_ARG;
    }
    if (!workspace || ((uintptr_t)workspace & 255u) != 0) return VPP_ERR_WORKSPACE;
    if (workspace_bytes < p->ws_bytes) return VPP_ERR_WORKSPACE;
    if (p->groups.empty()) return VPP_OK;  // nothing to do: every segment is empty

    hipStream_t stream = (hipStream_t)stream_ptr;
    char* ws = (char*)workspace;
    const size_t groups_bytes = p->groups.size() * sizeof(LaunchGroup);
    const size_t merges_bytes = p->merges.size() * sizeof(CombineSeg);
    if (p->table_bytes && upload == Upload::direct) {
        if (hipMemcpyAsync(ws, p->groups.data(), groups_bytes, hipMemcpyHostToDevice, stream) != hipSuccess ||
            (merges_bytes && hipMemcpyAsync(ws + groups_bytes, p->merges.data(), merges_bytes, hipMemcpyHostToDevice,
                                            stream) != hipSuccess))
            return VPP_ERR_HIP;
    } else if (p->table_bytes) {
        const int slot = p->next_slot;
        p->next_slot = (p->next_slot + 1) % STAGING_SLOTS;
        if (!p->staging_done[slot]) {
            if (hipEventCreateWithFlags(&p->staging_done[slot], hipEventDisableTiming) != hipSuccess)
                return VPP_ERR_HIP;
        }
        if (p->staging_pending[slot]) {
            if (hipEventSynchronize(p->staging_done[slot]) != hipSuccess) return VPP_ERR_HIP;
            p->staging_pending[slot] = false;
        }
        if (p->staging_cap[slot] < p->table_bytes) {
            if (p->staging[slot]) (void)hipHostFree(p->staging[slot]);
            p->staging[slot] = nullptr;
            p->staging_cap[slot] = 0;
            if (hipHostMalloc((void**)&p->staging[slot], p->table_bytes, hipHostMallocDefault) != hipSuccess)
                return VPP_ERR_HIP;
            p->staging_cap[slot] = p->table_bytes;
        }
        memcpy(p->staging[slot], p->groups.data(), groups_bytes);
        if (merges_bytes) memcpy(p->staging[slot] + groups_bytes, p->merges.data(), merges_bytes);
        if (hipMemcpyAsync(ws, p->staging[slot], p->table_bytes, hipMemcpyHostToDevice, stream) != hipSuccess)
            return VPP_ERR_HIP;
        if (hipEventRecord(p->staging_done[slot], stream) != hipSuccess) return VPP_ERR_HIP;
        p->staging_pending[slot] = true;
    }

    const vpp_chunk_attn_config_t& c = p->cfg;
    Launch l;  // of the tables only the entries in use are written
    memset(&l.a, 0, sizeof l.a);
    memset(&l.merge, 0, sizeof l.merge);
    l.nb = p->nb;
    l.dqk = c.head_dim_qk;
    l.nt = p->nt;
    l.workgroups = p->workgroups;
    AttnArgs& a = l.a;
    plan_args(p, a);
    if (p->table_bytes) a.groups = (const LaunchGroup*)ws;
    else memcpy(l.groups.g, p->groups.data(), groups_bytes);
    a.q = (const u16*)q;
    a.k = (const u16*)k;
    a.v = (const u16*)v;
    a.out = (u16*)out;
    a.lse = lse;
    a.part_o = (float*)(ws + p->part_o_off);
    a.part_lse = (float*)(ws + p->part_lse_off);
    a.q_st = (int32_t)q_st; a.q_sh = (int32_t)q_sh; a.k_st = (int32_t)k_st; a.k_sh = (int32_t)k_sh;
    a.v_st = (int32_t)v_st; a.v_sh = (int32_t)v_sh; a.o_st = (int32_t)o_st; a.o_sh = (int32_t)o_sh;
    a.lse_sh = (int32_t)lse_sh;
    if (rope) {
        a.k_rope = (const u16*)rope->k_rope;
        a.kr_st = (int32_t)rope->kr_st;
    }
    if (pg) {
        a.block_table = pg->block_table;
        a.bt_st = pg->bt_st;
        a.k_sp = pg->k_sp;
        a.v_sp = pg->v_sp;
        a.page_shift = pg->page_shift;
        a.num_pages = pg->num_pages;
    }
    if (!p->merges.empty()) {
        CombineArgs& m = l.merge;
        m.num_segs = (int32_t)p->merges.size();
        if (p->table_bytes) m.segs = (const CombineSeg*)(ws + groups_bytes);
        else memcpy(l.segs.s, p->merges.data(), merges_bytes);
        m.part_o = a.part_o;
        m.part_lse = a.part_lse;
        m.out = (u16*)out;
        m.lse = lse;
        m.o_st = o_st; m.o_sh = o_sh; m.lse_sh = lse_sh;
        m.num_heads = c.num_q_heads;
        m.blocks = p->merge_blocks;
    }
    const hipError_t e = rope ? vpp_detail::launch_attn_rope(l, stream)
                         : pg ? vpp_detail::launch_attn_paged(l, stream)
                              : vpp_detail::launch_attn_contig(l, stream);
    return e == hipSuccess ? VPP_OK : VPP_ERR_HIP;
}

}  // namespace

extern "C" vpp_status_t vpp_chunk_attn_run(vpp_chunk_attn_plan_t p, const void* q, int64_t q_st, int64_t q_sh,
                                           const void* k, int64_t k_st, int64_t k_sh, const void* v,
                                           int64_t v_st, int64_t v_sh, void* out, int64_t o_st, int64_t o_sh,
                                           float* lse, int64_t lse_sh, void* workspace, size_t workspace_bytes,
                                           void* stream_ptr) {
    return run_impl(p, q, q_st, q_sh, k, k_st, k_sh, v, v_st, v_sh, out, o_st, o_sh, lse, lse_sh, workspace,
                    workspace_bytes, stream_ptr, nullptr);
}

// ---------------------------------------------------------------------------
// No-allocation entry point. Its workspace is this file-scope device array (one
// copy per GPU, held until the process ends). In host code the name `scratch`
// is only a stand-in for the symbol, never a device address: the array's
// address on each device is looked up once, with that device current, and kept.
// ---------------------------------------------------------------------------
static __device__ __align__(256) char scratch[VPP_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void* scratch_addr[MAX_DEVICES] = {};

// The current device's copy of `scratch` (looked up on the first call on that device).
vpp_status_t scratch_on_current_device(void** addr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return VPP_ERR_HIP;
    if (dev >= MAX_DEVICES) return VPP_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_addr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return VPP_ERR_HIP;
        scratch_addr[dev] = ptr;
    }
    *addr = scratch_addr[dev];
    return VPP_OK;
}

}  // namespace

extern "C" vpp_status_t vpp_chunk_attn_run_noalloc(vpp_chunk_attn_plan_t p, const void* q, int64_t q_st,
                                                   int64_t q_sh, const void* k, int64_t k_st, int64_t k_sh,
                                                   const void* v, int64_t v_st, int64_t v_sh, void* out,
                                                   int64_t o_st, int64_t o_sh, float* lse, int64_t lse_sh,
                                                   void* stream_ptr) {
    if (!p) return VPP_ERR_INVALID_ARG;
    if (p->ws_bytes > (size_t)VPP_NOALLOC_SCRATCH_BYTES) return VPP_ERR_WORKSPACE;
    void* ws = nullptr;
    const vpp_status_t st = scratch_on_current_device(&ws);
    if (st != VPP_OK) return st;
    return run_impl(p, q, q_st, q_sh, k, k_st, k_sh, v, v_st, v_sh, out, o_st, o_sh, lse, lse_sh, ws,
                    (size_t)VPP_NOALLOC_SCRATCH_BYTES, stream_ptr, nullptr, nullptr, Upload::direct);
}

extern "C" vpp_status_t vpp_chunk_attn_run_mla(vpp_chunk_attn_plan_t p, const void* q, int64_t q_st,
                                               int64_t q_sh, const void* k_nope, int64_t kn_st, int64_t kn_sh,
                                               const void* k_rope, int64_t kr_st, const void* v, int64_t v_st,
                                               int64_t v_sh, void* out, int64_t o_st, int64_t o_sh, float* lse,
                                               int64_t lse_sh, void* workspace, size_t workspace_bytes,
                                               void* stream_ptr) {
    RopeK rope{k_rope, kr_st};
    return run_impl(p, q, q_st, q_sh, k_nope, kn_st, kn_sh, v, v_st, v_sh, out, o_st, o_sh, lse, lse_sh,
                    workspace, workspace_bytes, stream_ptr, nullptr, &rope);
}

extern "C" vpp_status_t vpp_chunk_attn_run_paged(vpp_chunk_attn_plan_t p, const void* q, int64_t q_st,
                                                 int64_t q_sh, const void* k_pages, int64_t k_sp, int64_t k_st,
                                                 int64_t k_sh, const void* v_pages, int64_t v_sp, int64_t v_st,
                                                 int64_t v_sh, int32_t page_size, int32_t num_pages,
                                                 const int32_t* block_table, int64_t bt_st, void* out,
                                                 int64_t o_st, int64_t o_sh, float* lse, int64_t lse_sh,
                                                 void* workspace, size_t workspace_bytes, void* stream_ptr) {
    if (!p || !block_table || ((uintptr_t)block_table & 3u) != 0) return VPP_ERR_INVALID_ARG;
    if (page_size < BN || page_size > (1 << 20) || (page_size & (page_size - 1)) != 0) return VPP_ERR_INVALID_ARG;
    if (num_pages < 1 || bt_st < 0) return VPP_ERR_INVALID_ARG;
    // pages start on 16-byte boundaries, and one page's rows fit the kernels' 32-bit row offsets
    if (!stride_ok(k_sp) || !stride_ok(v_sp) || k_sp < 1 || v_sp < 1) return VPP_ERR_INVALID_ARG;
    if ((int64_t)page_size * k_st >= ((int64_t)1 << 31) || (int64_t)page_size * v_st >= ((int64_t)1 << 31))
        return VPP_ERR_INVALID_ARG;
    for (const SegPlan& s : p->segs)
        if (s.kv_start % BN != 0) return VPP_ERR_INVALID_ARG;  // a key tile must not straddle two pages
    int shift = 0;
    while ((1 << shift) < page_size) ++shift;
    PagedKV pg{block_table, bt_st, k_sp, v_sp, shift, num_pages};
    return run_impl(p, q, q_st, q_sh, k_pages, k_st, k_sh, v_pages, v_st, v_sh, out, o_st, o_sh, lse, lse_sh,
                    workspace, workspace_bytes, stream_ptr, &pg);
}

extern "C" vpp_status_t vpp_kv_append_paged(const void* k_new, int64_t kn_st, int64_t kn_sh, const void* v_new,
                                            int64_t vn_st, int64_t vn_sh, void* k_pages, int64_t k_sp,
                                            int64_t k_st, int64_t k_sh, void* v_pages, int64_t v_sp, int64_t v_st,
                                            int64_t v_sh, int32_t num_tokens, int32_t num_kv_heads,
                                            int32_t head_dim_qk, int32_t head_dim_v, int32_t page_size,
                                            int32_t num_pages, const int64_t* slot_mapping, void* stream_ptr) {
    if (num_tokens < 0 || num_kv_heads < 1 || num_pages < 1) return VPP_ERR_INVALID_ARG;
    if (head_dim_qk < 8 || head_dim_v < 8 || head_dim_qk % 8 || head_dim_v % 8 || head_dim_qk > 1024 ||
        head_dim_v > 1024)
        return VPP_ERR_INVALID_ARG;
    if (page_size < BN || page_size > (1 << 20) || (page_size & (page_size - 1)) != 0) return VPP_ERR_INVALID_ARG;
    if (num_tokens == 0) return VPP_OK;
    if (!k_new || !v_new || !k_pages || !v_pages || !slot_mapping) return VPP_ERR_INVALID_ARG;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_pages) || !aligned16(v_pages) ||
        ((uintptr_t)slot_mapping & 7u) != 0)
        return VPP_ERR_INVALID_ARG;
    const int64_t st[] = {kn_st, kn_sh, vn_st, vn_sh, k_sp, k_st, k_sh, v_sp, v_st, v_sh};
    for (int64_t x : st)
        if (!stride_ok(x)) return VPP_ERR_INVALID_ARG;
    const int64_t total = (int64_t)num_tokens * num_kv_heads * ((head_dim_qk + head_dim_v) / 8);
    if (total >= ((int64_t)1 << 31) - 256) return VPP_ERR_INVALID_ARG;
    AppendArgs a;
    a.k_new = (const u16*)k_new;
    a.v_new = (const u16*)v_new;
    a.k_pages = (u16*)k_pages;
    a.v_pages = (u16*)v_pages;
    a.slots = slot_mapping;
    a.kn_st = kn_st; a.kn_sh = kn_sh; a.vn_st = vn_st; a.vn_sh = vn_sh;
    a.k_sp = k_sp; a.k_st = k_st; a.k_sh = k_sh; a.v_sp = v_sp; a.v_st = v_st; a.v_sh = v_sh;
    a.tokens = num_tokens;
    a.k_gran = head_dim_qk / 8;
    a.v_gran = head_dim_v / 8;
    a.k_token = num_kv_heads * a.k_gran;
    a.granules = num_kv_heads * (a.k_gran + a.v_gran);
    a.by_token = divisor((uint32_t)a.granules);
    a.by_k = divisor((uint32_t)a.k_gran);
    a.by_v = divisor((uint32_t)a.v_gran);
    int shift = 0;
    while ((1 << shift) < page_size) ++shift;
    a.page_shift = shift;
    a.num_pages = num_pages;
    // Non-temporal past 64 MB of new rows, twice the L2s: below, the rows stay cached for
    // the attention that follows.
    const bool nt = total * 16 > ((int64_t)64 << 20);
    auto* kernel = a.granules % 64 == 0 ? (nt ? kv_append_kernel<true, true> : kv_append_kernel<true, false>)
                                        : (nt ? kv_append_kernel<false, true> : kv_append_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream_ptr, a);
    return hipGetLastError() == hipSuccess ? VPP_OK : VPP_ERR_HIP;
}

extern "C" vpp_status_t vpp_paged_slot_mapping(int32_t num_segments, const int32_t* cu_q, const int64_t* kv_start,
                                               const int64_t* prefix_len, const int32_t* block_table,
                                               int64_t block_table_stride, int32_t pages_per_row,
                                               int32_t page_size, int64_t* slot_mapping) {
    if (num_segments < 0 || !cu_q || page_size < 1 || pages_per_row < 0 || block_table_stride < 0)
        return VPP_ERR_INVALID_ARG;
    if (num_segments == 0) return VPP_OK;
    if (!kv_start || !prefix_len || !block_table || !slot_mapping || cu_q[0] != 0) return VPP_ERR_INVALID_ARG;
    for (int s = 0; s < num_segments; ++s) {
        if (cu_q[s + 1] < cu_q[s] || kv_start[s] < 0 || prefix_len[s] < 0) return VPP_ERR_INVALID_ARG;
        for (int r = cu_q[s]; r < cu_q[s + 1]; ++r) {
            const int64_t row = kv_start[s] + prefix_len[s] + (r - cu_q[s]);
            const int64_t idx = row / page_size;
            if (idx >= pages_per_row) return VPP_ERR_INVALID_ARG;
            const int32_t pg = block_table[(int64_t)s * block_table_stride + idx];
            if (pg < 0) return VPP_ERR_INVALID_ARG;
            slot_mapping[r] = (int64_t)pg * page_size + row % page_size;
        }
    }
    return VPP_OK;
}

#endif  // host code (part 0)
