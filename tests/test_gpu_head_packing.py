"""Query tiles that hold several heads of one kv head (GQA), against the fp64 oracle.

A tile's rows are (token, head) pairs: the largest divisor of Hq/Hkv up to 16 heads, and as
many tokens as fit 128 or 256 rows. Group sizes that do and do not divide the tile, and
segment lengths one below, at and one above a tile's tokens, unsplit and split.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import parity as PA

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rand(shape, std, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=DEV) * std).to(torch.bfloat16)


def _pack(hq, hkv):
    return max(n for n in range(1, 17) if (hq // hkv) % n == 0)


@pytest.mark.parametrize("nb", [1, 2])
@pytest.mark.parametrize("hq,hkv,dims", [
    (8, 2, (128, 128)),      # 4 heads a tile
    (5, 1, (64, 64)),        # 5: 255 of 256 rows, 125 of 128
    (14, 2, (128, 128)),     # 7
    (16, 1, (64, 64)),       # 16
    (17, 1, (64, 64)),       # 17 has no divisor up to 16: one head a tile
    (24, 1, (128, 128)),     # 24 heads: two tiles of 12
    (6, 2, (192, 128)),      # 3
])
@pytest.mark.parametrize("splits", [1, 2])
def test_packed_heads(hq, hkv, dims, nb, splits, monkeypatch):
    from paper_2608_26523_amd.attention import ChunkAttention
    monkeypatch.setenv("VPP_NB", str(nb))
    dqk, dv = dims
    tt = 128 * nb // _pack(hq, hkv)
    segs = [(0, tt - 1), (130, tt), (67, tt + 1), (200, 2 * tt + 1), (0, 1), (64, 3)]  # (prefix, rows)
    kvs = [int(x) for x in np.cumsum([0] + [p + n for p, n in segs[:-1]])]
    T = sum(p + n for p, n in segs)
    cu = np.cumsum([0] + [n for _, n in segs])
    tok = int(cu[-1])
    print("case:", hq, hkv, dims, "nb", nb, "splits", splits, "tokens a tile", tt, flush=True)
    std = 1.0 / math.sqrt(dqk)
    q, k, v = _rand((tok, hq, dqk), 1.0, 1), _rand((T, hkv, dqk), std, 2), _rand((T, hkv, dv), std, 3)
    attn = ChunkAttention(hq, hkv, dqk, dv, max_chunk_tokens=tok, max_kv_len=T, num_splits=splits)
    out, lse = PA.run_chunk(attn, q, k, v, cu, kvs, [p for p, _ in segs])
    assert attn.info().block_m == 128 * nb
    ro, rl = oracle.attention_full(q.cpu(), k.cpu(), v.cpu(), cu, kvs, [p for p, _ in segs])
    r, h = np.repeat(np.arange(tok), hq), np.tile(np.arange(hq), tok)
    rep = PA.compare(out, lse, r, h, ro.reshape(tok * hq, -1), rl.T.reshape(-1))
    assert rep.ok(), str(rep)
