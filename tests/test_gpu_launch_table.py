"""Chunks of many segments: the launch table around its limits, against the fp64 oracle.

A run's launch table has one entry per segment that has rows. Up to 64
entries travel in the kernel arguments, more are copied to the workspace; a workgroup finds
its entry by comparing 64 at a time, so 64/65 and 4096/4097 are where the search takes
another step. Segments without a prefix have one piece whatever the split count and write
their results directly, next to split segments whose partials are merged.
"""
import numpy as np
import pytest
import torch

import oracle
import parity as PA

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rand(shape, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=DEV) / 8.0).to(torch.bfloat16)


# (segments, rows of every second segment, prefix of every third, heads, split request)
@pytest.mark.parametrize("nseg,rows,prefix,heads,splits", [
    (64, 3, 0, (4, 2), 1),
    (65, 3, 0, (4, 2), 1),
    (33, 5, 130, (3, 1), 2),     # 11 merged segments
    (60, 2, 200, (4, 4), 3),     # 20 merged segments
    (200, 1, 140, (2, 1), 2),    # 67 merged segments
    (4096, 1, 0, (1, 1), 1),
    (4097, 1, 0, (2, 1), 1),
    (3, 300, 700, (4, 2), -1),
])
def test_many_segments(nseg, rows, prefix, heads, splits):
    from paper_2608_26523_amd.attention import ChunkAttention
    hq, hkv = heads
    lens = [rows if i % 2 else 1 for i in range(nseg)]
    pre = [prefix if i % 3 == 0 else 0 for i in range(nseg)]
    kvs, at = [], 0
    for n, p in zip(lens, pre):
        kvs.append(at)
        at += n + p
    cu = np.cumsum([0] + lens)
    tok = int(cu[-1])
    print("case:", nseg, rows, prefix, heads, splits, flush=True)
    q, k, v = _rand((tok, hq, 64), 1), _rand((at, hkv, 64), 2), _rand((at, hkv, 64), 3)
    attn = ChunkAttention(hq, hkv, 64, 64, max_chunk_tokens=tok, max_kv_len=at, max_segments=nseg,
                          num_splits=splits)
    out, lse = PA.run_chunk(attn, q, k, v, cu, kvs, pre)
    ro, rl = oracle.attention_full(q.cpu(), k.cpu(), v.cpu(), cu, kvs, pre)
    r, h = np.repeat(np.arange(tok), hq), np.tile(np.arange(hq), tok)
    rep = PA.compare(out, lse, r, h, ro.reshape(tok * hq, -1), rl.T.reshape(-1))
    assert rep.ok(), str(rep)
    # the entry point without a workspace, whose table copy is synchronous
    out2, lse2 = torch.full_like(out, -3.0), torch.full_like(lse, -3.0)
    attn.run_noalloc(q, k, v, out2, lse2)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


# pieces per segment: 2, 5, 9, 16 (the merge walks them one, two, four and eight ways), and
# automatic plans of few rows behind long prefixes, whose segments are cut each on its own
@pytest.mark.parametrize("heads,dims,segs,splits", [
    ((4, 2), (128, 128), [(2000, 37)], 2),
    ((4, 2), (128, 128), [(2000, 37), (300, 5)], 5),
    ((3, 3), (64, 64), [(2000, 37), (70, 9)], 9),
    ((2, 2), (192, 128), [(2000, 37), (0, 200)], 16),
    ((4, 4), (64, 64), [(20000, 3)], -1),
    ((4, 1), (128, 128), [(9000, 217), (40, 300)], -1),
    ((8, 2), (128, 128), [(6000, 40), (3000, 1), (0, 700), (100, 1)], -1),
    ((16, 16), (192, 128), [(5000, 60), (700, 1)], -1),
    # few head groups and long last pieces: launched as two runs
    ((4, 1), (128, 128), [(200, 600)], 3),
    ((9, 9), (64, 64), [(130, 300)], 2),
    ((3, 1), (192, 128), [(256, 500), (64, 90), (900, 40)], 4),
])
def test_pieces_and_merge(heads, dims, segs, splits):
    from paper_2608_26523_amd.attention import ChunkAttention
    (hq, hkv), (dqk, dv) = heads, dims
    kvs = [int(x) for x in np.cumsum([0] + [p + n for p, n in segs[:-1]])]
    T = sum(p + n for p, n in segs)
    cu = np.cumsum([0] + [n for _, n in segs])
    tok = int(cu[-1])
    print("case:", heads, dims, segs, splits, flush=True)
    q, k, v = _rand((tok, hq, dqk), 1), _rand((T, hkv, dqk), 2), _rand((T, hkv, dv), 3)
    attn = ChunkAttention(hq, hkv, dqk, dv, max_chunk_tokens=tok, max_kv_len=T, num_splits=splits)
    out, lse = PA.run_chunk(attn, q, k, v, cu, kvs, [p for p, _ in segs])
    assert attn.info().num_splits == splits if splits > 0 else attn.info().num_splits > 1
    ro, rl = oracle.attention_full(q.cpu(), k.cpu(), v.cpu(), cu, kvs, [p for p, _ in segs])
    r, h = np.repeat(np.arange(tok), hq), np.tile(np.arange(hq), tok)
    rep = PA.compare(out, lse, r, h, ro.reshape(tok * hq, -1), rl.T.reshape(-1))
    assert rep.ok(), str(rep)


# single tokens behind cached prefixes: one tile a head group, whose K/V copies are
# non-temporal; contiguous against the oracle, paged and split keys against contiguous
@pytest.mark.parametrize("heads,dims", [((4, 2), (64, 64)), ((32, 4), (128, 128)), ((6, 6), (192, 128))])
def test_single_tokens(heads, dims):
    from paper_2608_26523_amd.attention import ChunkAttention
    (hq, hkv), (dqk, dv) = heads, dims
    pre, page = [0, 63, 64, 700, 5000], 64
    n = len(pre)
    rows = [p + 1 for p in pre]
    kvs = [int(x) for x in np.cumsum([0] + rows[:-1])]
    cu = np.arange(n + 1)
    T = sum(rows)
    print("case:", heads, dims, flush=True)
    q, k, v = _rand((n, hq, dqk), 1), _rand((T, hkv, dqk), 2), _rand((T, hkv, dv), 3)
    if dqk == 192:
        k[:, 1:, 128:] = k[:, :1, 128:]  # one shared part per row
    attn = ChunkAttention(hq, hkv, dqk, dv, max_chunk_tokens=n, max_kv_len=T)
    out, lse = PA.run_chunk(attn, q, k, v, cu, kvs, pre)
    assert attn.info().block_m == 128
    ro, rl = oracle.attention_full(q.cpu(), k.cpu(), v.cpu(), cu, kvs, pre)
    r, h = np.repeat(np.arange(n), hq), np.tile(np.arange(hq), n)
    rep = PA.compare(out, lse, r, h, ro.reshape(n * hq, -1), rl.T.reshape(-1))
    assert rep.ok(), str(rep)
    if dqk == 192:
        out_s, _ = attn.run_mla(q, k[:, :, :128], k[:, 0, 128:], v)
        assert torch.equal(out_s, out)
    per = [-(-x // page) for x in rows]
    table = torch.zeros((n, max(per)), dtype=torch.int32)
    kp = torch.zeros((sum(per), page, hkv, dqk), dtype=torch.bfloat16, device=DEV)
    vp = torch.zeros((sum(per), page, hkv, dv), dtype=torch.bfloat16, device=DEV)
    at = 0
    for s in range(n):
        table[s, :per[s]] = torch.arange(at, at + per[s])
        kp[at:at + per[s]].view(-1, hkv, dqk)[:rows[s]] = k[kvs[s]:kvs[s] + rows[s]]
        vp[at:at + per[s]].view(-1, hkv, dv)[:rows[s]] = v[kvs[s]:kvs[s] + rows[s]]
        at += per[s]
    attn.plan(cu, [0] * n, pre)
    out_p, _ = attn.run_paged(q, kp, vp, table.to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(out_p, out)


@pytest.mark.parametrize("pieces", [2, 3, 5, 7, 9, 11, 16])
def test_merge_keeps_infinities(pieces):
    """An infinite V in the first piece (a key every row sees) gives that column's infinity, as
    it does without a split, and leaves every other column as it is: the merge reads nothing past
    a row's last piece, whatever the lane group's four places in flight hold."""
    from paper_2608_26523_amd.attention import ChunkAttention
    hq, hkv, d, n, p = 4, 2, 64, 5, 64 * 17
    print("case:", pieces, flush=True)
    q, k, v = _rand((n, hq, d), 1), _rand((n + p, hkv, d), 2), _rand((n + p, hkv, d), 3)
    got = []
    for splits in (1, pieces):
        attn = ChunkAttention(hq, hkv, d, d, max_chunk_tokens=n, max_kv_len=n + p, num_splits=splits)
        assert attn.plan([0, n], [0], [p]).num_splits == splits
        res = []
        for inf in (False, True):
            x = v.clone()
            if inf:
                x[3, :, 7], x[3, :, 40] = float("inf"), -float("inf")
            out, _ = attn.run(q, k, x, torch.empty((n, hq, d), dtype=torch.bfloat16, device=DEV))
            torch.cuda.synchronize()
            res.append(out.float())
        got.append(res)
    for plain, inf in got:
        plain[..., 7], plain[..., 40] = float("inf"), -float("inf")
        assert torch.equal(plain, inf)


@pytest.mark.parametrize("pieces", [2, 5, 16])
def test_merge_of_rows_without_weight(pieces):
    """Rows whose every score is -inf give zeros and lse -inf, split as unsplit: no piece of
    such a row has any weight."""
    from paper_2608_26523_amd.attention import ChunkAttention
    hq, hkv, d, n, p = 4, 2, 64, 5, 64 * 17
    print("case:", pieces, flush=True)
    q, k, v = _rand((n, hq, d), 1), _rand((n + p, hkv, d), 2), _rand((n + p, hkv, d), 3)
    q[:, 1], k[:, 0] = 1.0, -float("inf")  # head 1 (kv head 0)
    q[:, 0] = 0.5                          # head 0 reads the same keys
    got = []
    for splits in (1, pieces):
        attn = ChunkAttention(hq, hkv, d, d, max_chunk_tokens=n, max_kv_len=n + p, num_splits=splits)
        assert attn.plan([0, n], [0], [p]).num_splits == splits
        out = torch.empty((n, hq, d), dtype=torch.bfloat16, device=DEV)
        lse = torch.empty((hq, n), dtype=torch.float32, device=DEV)
        attn.run(q, k, v, out, lse)
        torch.cuda.synchronize()
        got.append((out, lse))
    for out, lse in got:
        assert (out[:, :2] == 0).all() and (lse[:2] == -float("inf")).all()
        assert torch.isfinite(out[:, 2:].float()).all() and torch.isfinite(lse[2:]).all()
