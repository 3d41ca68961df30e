"""Every workgroup of a planned launch, replayed on the CPU (no GPU).

``launch_replay.hip`` is the library's host code without its kernels, and calls the functions by
which the kernels find their table entry, tiles, keys, results and merge pairs. For each plan:

* the grid is the table's own workgroups, and each finds the entry that it belongs to;
* the tiles of a segment cover each of its rows once per head and piece, and lie in it;
* the pieces of a tile follow each other from key 0 to the tile's last position;
* results go to the tile's own chunk rows, or to partial rows that no other (segment, piece) has
  and that lie in the workspace;
* the merge takes each (row, head) of each split segment once in each of its ways;
* the tiles are those of plan_items with keys, once per head group, so that the replay of the
  copies of listed tiles (test_kernel_bounds_cpu.py) holds for what is launched.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2608_26523_amd import binding as B
from paper_2608_26523_amd import build as Bld
from paper_2608_26523_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
BLOCK, ENTRY, SUB, H, HK, ROW0, NROWS, POS0, KB, KE, OUT = range(11)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("replay") / "launch_replay.so")
    res = subprocess.run([Bld.hipcc()] + Bld.HIPCC_FLAGS + ["-I", Bld.INCLUDE, "-o", out,
                                                            os.path.join(HERE, "launch_replay.hip")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    x = B.load(out)
    vp = ctypes.c_void_p
    for name, args, ret in (("replay_summary", [vp, vp], None), ("replay_groups", [vp, vp], None),
                            ("replay_merges", [vp, vp], None), ("replay_tiles", [vp, vp], ctypes.c_int64),
                            ("replay_merge", [vp, vp], ctypes.c_int64), ("replay_key_bytes", [vp], ctypes.c_double)):
        getattr(x, name).argtypes, getattr(x, name).restype = args, ret
    return x


class Replay:
    def __init__(self, lib, hq, hkv, dqk, dv, lens, pre, splits=-1, kvs=None):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        kv = np.array(kvs if kvs is not None else [0] * len(lens), dtype=np.int64)
        pl = np.array(pre, dtype=np.int64)
        cfg = B.Config(num_q_heads=hq, num_kv_heads=hkv, head_dim_qk=dqk, head_dim_v=dv, softmax_scale=0.0, causal=1,
                       max_chunk_tokens=max(int(cu[-1]), 1), max_segments=len(lens), max_kv_len=1 << 30,
                       num_splits=splits)
        h, ws = ctypes.c_void_p(None), ctypes.c_size_t(0)
        st = lib.vpp_chunk_attn_plan(ctypes.byref(cfg), len(lens), cu.ctypes.data, kv.ctypes.data, pl.ctypes.data,
                                     ctypes.byref(h), ctypes.byref(ws))
        assert st == B.VPP_OK
        self.cu, self.kv, self.pre, self.heads, self.dv = cu, kv, pl, (hq, hkv), dv
        s = np.zeros(12, dtype=np.int64)
        lib.replay_summary(h, s.ctypes.data)
        (self.workgroups, self.merge_blocks, ng, nm, self.part_o, self.part_lse, self.ws, self.table, self.pack, self.tt,
         self.head_groups, self.nt) = (int(x) for x in s)
        assert self.ws == ws.value
        self.groups, self.merges = np.zeros((ng, 10), dtype=np.int32), np.zeros((nm, 5), dtype=np.int32)
        lib.replay_groups(h, self.groups.ctypes.data)
        lib.replay_merges(h, self.merges.ctypes.data)
        tiles = np.zeros((2 * self.workgroups, 11), dtype=np.int32)
        self.tiles = tiles[:lib.replay_tiles(h, tiles.ctypes.data)]
        pairs = np.zeros((self.merge_blocks * (1024 // dv), 3), dtype=np.int64)
        self.pairs = pairs[:lib.replay_merge(h, pairs.ctypes.data)]
        self.key_bytes = lib.replay_key_bytes(h)
        n = ctypes.c_int32(0)
        assert lib.vpp_chunk_attn_plan_items(h, None, 0, ctypes.byref(n)) == B.VPP_OK
        self.items = np.zeros(n.value, dtype=B.WORK_ITEM_DTYPE)
        if n.value:
            assert lib.vpp_chunk_attn_plan_items(h, self.items.ctypes.data, n.value, ctypes.byref(n)) == B.VPP_OK
        lib.vpp_chunk_attn_destroy(h)


def _once(rows):
    """Whether no row occurs twice."""
    return len(np.unique(rows, axis=0)) == len(rows)


def _intervals_disjoint(begin, length):
    order = np.argsort(begin)
    return (begin[order][1:] >= (begin + length)[order][:-1]).all()


def check(lib, hq, hkv, dqk, dv, lens, pre, splits=-1, kvs=None):
    r = Replay(lib, hq, hkv, dqk, dv, lens, pre, splits, kvs)
    t, g = r.tiles, r.groups
    wg0, row0, length, prefix, kv_start, seg, pieces, part0, slots, ntiles = g.T.astype(np.int64)
    pieces = abs(pieces)  # negative: the last pieces are a run of their own
    # the table: one entry per segment with rows
    assert sorted(seg) == [s for s in range(len(lens)) if lens[s] > 0]
    assert (row0 == r.cu[seg]).all() and (length == np.diff(r.cu)[seg]).all()
    assert (prefix == r.pre[seg]).all() and (kv_start == r.kv[seg]).all()
    assert (ntiles == -(-length // r.tt)).all() and ((slots == ntiles) | (slots == (ntiles + 1) // 2)).all()
    assert r.pack * r.head_groups == hq and (hq // hkv) % r.pack == 0
    # the grid, and every workgroup's entry
    sizes = slots * pieces * r.head_groups
    assert (wg0 == np.cumsum(sizes) - sizes).all() and r.workgroups == sizes.sum()
    first = t[t[:, SUB] == 0]
    assert (first[:, BLOCK] == np.arange(r.workgroups)).all()
    assert (first[:, ENTRY] == np.searchsorted(wg0, first[:, BLOCK], side="right") - 1).all()
    # tiles: rows, heads, keys
    e = t[:, ENTRY]
    ti = (t[:, ROW0] - row0[e]) // r.tt
    assert (ti >= 0).all() and (ti < ntiles[e]).all() and (t[:, ROW0] == row0[e] + ti * r.tt).all()
    assert (t[:, NROWS] == np.minimum(r.tt, length[e] - ti * r.tt)).all() and (t[:, POS0] == prefix[e] + ti * r.tt).all()
    assert (t[:, H] % r.pack == 0).all() and (t[:, H] + r.pack <= hq).all() and (t[:, HK] == t[:, H] // (hq // hkv)).all()
    assert (0 <= t[:, KB]).all() and (t[:, KB] < t[:, KE]).all() and (t[:, KE] <= t[:, POS0] + t[:, NROWS]).all()
    # pieces of a (segment, tile, head group) in key order: from 0 to the last position, end to begin
    order = np.lexsort((t[:, KB], t[:, H], ti, e))
    s = t[order]
    key = np.stack([e[order], ti[order], s[:, H]], axis=1)
    starts = np.concatenate([[True], (key[1:] != key[:-1]).any(axis=1)]) if len(s) else np.zeros(0, dtype=bool)
    ends = np.concatenate([starts[1:], [True]]) if len(s) else starts
    assert starts.sum() == (ntiles * r.head_groups).sum() and len(s) == (ntiles * r.head_groups * pieces).sum()
    assert (s[starts, KB] == 0).all() and (s[ends, KE] == s[ends, POS0] + s[ends, NROWS]).all()
    assert (s[1:][~starts[1:], KB] == s[:-1][~ends[:-1], KE]).all()
    # results: chunk rows, or partial rows piece by piece
    split = pieces[e] > 1
    assert (t[~split, OUT] == t[~split, ROW0]).all() and (t[split, OUT] < 0).all()
    assert ((part0 >= 0) == (pieces > 1)).all()
    part = ~t[split, OUT].astype(np.int64)
    one = t[split, H] == 0
    total = int((pieces * length)[pieces > 1].sum())
    assert _intervals_disjoint(part[one], t[split, NROWS][one]) and int(t[split, NROWS][one].sum()) == total
    assert _once(np.stack([part, t[split, H]], axis=1))
    assert (part >= 0).all() and (part + t[split, NROWS] <= total).all()
    assert r.table <= r.part_o and r.part_o % 16 == 0 and r.part_o + total * hq * dv * 4 <= r.part_lse
    assert r.part_lse % 16 == 0 and r.part_lse + total * hq * 4 <= r.ws
    assert r.table == (40 * len(g) + 20 * len(r.merges) if len(g) > 64 else 0)
    # piece b of a split segment's row i is partial row part0 + b * len + i, as the merge reads it
    b = (part - part0[e[split]] - ti[split] * r.tt) // length[e[split]]
    assert (part == part0[e[split]] + b * length[e[split]] + ti[split] * r.tt).all()
    assert (b >= 0).all() and (b < pieces[e[split]]).all()
    # the merge: the split segments, each pair once a way
    merged = np.stack([row0, length, pieces, part0], axis=1)[pieces > 1]
    assert (r.merges[:, 1:] == merged).all()
    assert _once(r.pairs)
    ways = np.array([lib.replay_merge_ways(int(n)) for n in r.merges[:, 3]], dtype=np.int64)
    assert len(r.pairs) == (ways * r.merges[:, 2].astype(np.int64) * hq).sum()
    if len(r.pairs):
        m = r.pairs[:, 0]
        assert (r.pairs[:, 1] < r.merges[m, 2].astype(np.int64) * hq).all() and (r.pairs[:, 2] < ways[m]).all()
    # plan_items lists the same tiles
    it = r.items[(r.items["nrows"] > 0) & (r.items["key_end"] > r.items["key_begin"])]
    listed = np.stack([it[f] for f in ("row0", "nrows", "pos0", "key_begin", "key_end", "kv_base")], axis=1)
    for h in {0, hq - r.pack}:
        x = t[t[:, H] == h]
        run = np.concatenate([x[:, [ROW0, NROWS, POS0, KB, KE]], kv_start[x[:, ENTRY]][:, None]], axis=1)
        assert len(run) == len(listed) and (run[np.lexsort(run.T)] == listed[np.lexsort(listed.T)]).all()
    return r


@pytest.mark.parametrize("name", ["tiny", "gqa", "mla", "long"])
def test_workload_chunks(lib, name):
    w = W.get(name)
    for k in sorted({0, 1, W.num_chunks(w) // 2, W.num_chunks(w) - 1}):
        _, cu, kvs, pre = W.chunk_segments(w, k)
        check(lib, w.hq, w.hkv, w.dqk, w.dv, list(np.diff(cu)), pre, w.num_splits, kvs)


def test_mixed_chunks(lib):
    w = W.get("mixed")
    n = W.num_chunks(w)
    for k in list(range(0, n, 29)) + [n - 1]:
        _, cu, kvs, pre = W.chunk_segments(w, k)
        check(lib, w.hq, w.hkv, w.dqk, w.dv, list(np.diff(cu)), pre, w.num_splits, kvs)


@pytest.mark.parametrize("seed", range(80))
def test_random_plans(lib, seed):
    rng = np.random.default_rng(seed)
    n = int(rng.choice([1, 2, 5, 40, 64, 65, 200]))
    top = 3000 if n <= 5 else 60
    lens = [int(rng.integers(0, top)) if rng.random() > 0.1 else 0 for _ in range(n)]
    lens[int(rng.integers(n))] = 1 + int(rng.integers(0, 700))
    pre = [int(rng.choice([0, rng.integers(0, 100), rng.integers(0, 5000), rng.integers(0, 60000)])) for _ in range(n)]
    hq, hkv = [(4, 4), (8, 2), (2, 1), (16, 16), (64, 4), (32, 1), (17, 1), (24, 2), (71, 1), (5, 5), (12, 1)][int(rng.integers(11))]
    dqk, dv = [(64, 64), (128, 128), (192, 128)][int(rng.integers(3))]
    check(lib, hq, hkv, dqk, dv, lens, pre, int(rng.choice([-1, -1, 1, 2, 5, 16])), [64 * i for i in range(n)])


@pytest.mark.parametrize("nseg", [64, 65, 4096, 4097])
def test_table_search_steps(lib, nseg):
    check(lib, 2, 1, 64, 64, [1] * nseg, [0 if i % 7 else 130 for i in range(nseg)], 2)


@pytest.mark.parametrize("remap", ["0", "1"])
def test_workgroup_order(lib, remap, monkeypatch):
    monkeypatch.setenv("VPP_XCD_REMAP", remap)
    check(lib, 6, 2, 128, 128, [3000, 40], [0, 20000], 3)
    check(lib, 32, 8, 128, 128, [700, 1, 129], [9000, 64, 63])


def test_empty_chunk(lib):
    r = Replay(lib, 4, 2, 64, 64, [0, 0], [3, 0])
    assert r.workgroups == 0 and r.merge_blocks == 0 and len(r.tiles) == 0


def test_row_token_is_the_division(lib):
    for pack in range(1, 17):
        for row in range(256):
            assert lib.replay_row_token(row, pack) == row // pack


# heads per kv head: 1, 4, 16 fit one tile; 17, 24, 32 and 71 take several, which read the same keys
@pytest.mark.parametrize("hq,hkv,one_tile", [(16, 16, True), (32, 8, True), (64, 4, True), (4, 1, True), (17, 1, False),
                                             (34, 2, False), (24, 1, False), (64, 2, False), (71, 1, False)])
@pytest.mark.parametrize("dqk,dv", [(64, 64), (128, 128), (192, 128)])
def test_keys_read_by_one_workgroup(lib, hq, hkv, one_tile, dqk, dv):
    """Non-temporal copies only of keys that one workgroup reads, and every kv head's keys counted once."""
    lens, pre = [1] * 32, [4096 + 600 * i for i in range(32)]
    r = check(lib, hq, hkv, dqk, dv, lens, pre)
    t = r.tiles
    readers = np.unique(np.stack([t[:, ENTRY], t[:, HK], t[:, KB]], axis=1), axis=0, return_counts=True)[1]
    assert r.nt == one_tile == (readers.max() == 1)
    assert r.key_bytes == (sum(pre) + sum(lens)) * hkv * (dqk + dv) * 2


# few head groups: rows of one segment in fixed pieces, whose last piece is long (its own keys)
@pytest.mark.parametrize("hq,hkv,dqk,dv,rows,pre,splits", [
    (4, 1, 128, 128, 6089, 1539, 8), (4, 1, 128, 128, 6089, 1539, 16), (16, 1, 64, 64, 4000, 2000, 4),
    (8, 2, 128, 128, 5000, 1000, 4), (3, 3, 64, 64, 3000, 700, 5), (9, 9, 64, 64, 3000, 700, 4),
])
def test_long_pieces_are_spread_over_the_xcds(lib, hq, hkv, dqk, dv, rows, pre, splits):
    r = check(lib, hq, hkv, dqk, dv, [rows], [pre], splits)
    assert abs(r.groups[0, 6]) == splits
    steps = -(-(r.tiles[:, KE] - r.tiles[:, KB]) // 64).astype(np.int64)
    load = np.bincount(r.tiles[:, BLOCK] & 7, weights=steps, minlength=8)
    assert load.max() <= 1.25 * load.mean()
