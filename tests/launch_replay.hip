// Replays a planned launch on the CPU: the host code of the library, and the functions by
// which the kernels work out what each workgroup does, called for every workgroup.
#define VPP_PART 4
#include "../paper_2608_26523_amd/csrc/vpp_chunk_attn.hip"

// the kernels are not part of this build
hipError_t vpp_detail::launch_attn_contig(const Launch&, hipStream_t) { return hipErrorNotSupported; }
hipError_t vpp_detail::launch_attn_paged(const Launch&, hipStream_t) { return hipErrorNotSupported; }
hipError_t vpp_detail::launch_attn_rope(const Launch&, hipStream_t) { return hipErrorNotSupported; }

namespace {

// find_entry with the 64 lanes in a loop
template <typename First>
int find_on_host(int n, int x, First&& first) {
    EntrySearch e{0, n};
    while (e.cnt > 1) {
        int hits = 0;
        for (int lane = 0; lane < 64; ++lane) hits += e.has(lane) && first(e.entry(lane)) <= x;
        e.take(hits);
    }
    return e.lo;
}

}  // namespace

// workgroups, merge blocks, groups, merges,
// part_o_off, part_lse_off, workspace bytes, table bytes, pack, tile tokens, head groups, nt
extern "C" void replay_summary(vpp_chunk_attn_plan_t p, int64_t* out) {
    AttnArgs a{};
    plan_args(p, a);
    const int64_t v[] = {p->workgroups, p->merge_blocks, (int64_t)p->groups.size(), (int64_t)p->merges.size(),
                         (int64_t)p->part_o_off, (int64_t)p->part_lse_off, (int64_t)p->ws_bytes, (int64_t)p->table_bytes,
                         a.pack, a.tile_tokens, a.head_groups, p->nt};
    std::copy(std::begin(v), std::end(v), out);
}

// One row of 10 numbers per table entry: LaunchGroup's fields in order.
extern "C" void replay_groups(vpp_chunk_attn_plan_t p, int32_t* out) {
    static_assert(sizeof(LaunchGroup) == 40, "ten fields");
    memcpy(out, p->groups.data(), p->groups.size() * sizeof(LaunchGroup));
}

// One row of 5 numbers per merged segment: CombineSeg's fields in order.
extern "C" void replay_merges(vpp_chunk_attn_plan_t p, int32_t* out) {
    static_assert(sizeof(CombineSeg) == 20, "five fields");
    memcpy(out, p->merges.data(), p->merges.size() * sizeof(CombineSeg));
}

// One row of 11 numbers per tile of every workgroup: workgroup, table entry, sub, then
// TileWork's fields. Returns their count (capacity: two per workgroup).
extern "C" int64_t replay_tiles(vpp_chunk_attn_plan_t p, int32_t* out) {
    AttnArgs a{};
    plan_args(p, a);
    const TileArgs t{a.group, a.pack, a.tile_tokens, a.head_groups, a.xcd_remap};
    int64_t n = 0;
    for (int block = 0; block < p->workgroups; ++block) {
        const int e = find_on_host(a.num_groups, block, [&](int i) { return p->groups.at((size_t)i).wg0; });
        const LaunchGroup& g = p->groups.at((size_t)e);
        for (int sub = 0; sub < 2; ++sub) {
            TileWork w;
            if (!tile_work(t, g, block - g.wg0, sub, w)) break;
            const int32_t row[] = {block, e, sub, w.h, w.hk, w.row0, w.nrows, w.pos0, w.key_begin, w.key_end, w.out_row0};
            std::copy(std::begin(row), std::end(row), out + 11 * n++);
        }
    }
    return n;
}

// One row of 3 numbers per lane group of every merge block with a pair: merged segment, pair,
// way. Returns their count (capacity: 1024 / dv per block).
extern "C" int64_t replay_merge(vpp_chunk_attn_plan_t p, int64_t* out) {
    const int groups = 256 / (p->cfg.head_dim_v / 4);
    int64_t n = 0;
    for (int block = 0; block < p->merge_blocks; ++block) {
        const int e = find_on_host((int)p->merges.size(), block, [&](int i) { return p->merges.at((size_t)i).block0; });
        const CombineSeg& s = p->merges.at((size_t)e);
        for (int grp = 0; grp < groups; ++grp) {
            int way;
            const int64_t pair = merge_place(block - s.block0, groups, grp, merge_ways(s.pieces), way);
            if (pair >= (int64_t)s.len * p->cfg.num_q_heads) continue;
            out[3 * n] = e, out[3 * n + 1] = pair, out[3 * n + 2] = way;
            ++n;
        }
    }
    return n;
}

extern "C" int replay_row_token(int r, int pack) { return row_token(r, (65536 + pack - 1) / pack); }
extern "C" int replay_merge_ways(int pieces) { return merge_ways(pieces); }
extern "C" double replay_key_bytes(vpp_chunk_attn_plan_t p) { return launch_model(p->cfg, p->pack).key_bytes(p->segs); }
