"""Plans that run_noalloc's 64 MiB scratch took stay within it (host only).

The former workspace: 32 bytes per entry of one-head tiles (128 or 256 rows) run in pairs, and
the fp32 partials of every row for a split count common to the chunk. Fixed counts: the
workspace must not exceed that. Automatic ones: chunks that the former rule left unsplit, many
equal slots, must not need the scratch's size in partials.
"""
import numpy as np
import pytest

from paper_2608_26523_amd import binding as B


def _plan(hq, hkv, dqk, dv, lens, pre, splits):
    cu = np.concatenate([[0], np.cumsum(lens)])
    cfg = B.Config(num_q_heads=hq, num_kv_heads=hkv, head_dim_qk=dqk, head_dim_v=dv, softmax_scale=0.0, causal=1,
                   max_chunk_tokens=int(cu[-1]), max_segments=len(lens), max_kv_len=1 << 30, num_splits=splits)
    h, ws = B.vpp_chunk_attn_plan(cfg, cu, [0] * len(lens), pre)
    info = B.vpp_chunk_attn_plan_info(h)
    B.vpp_chunk_attn_destroy(h)
    return ws, info


def _a(x):
    return -(-int(x) // 256) * 256


@pytest.mark.parametrize("splits", [2, 3, 7, 16])
@pytest.mark.parametrize("hq,hkv,dqk,dv", [(64, 4, 128, 128), (16, 16, 192, 128), (4, 4, 64, 64), (5, 1, 64, 64)])
@pytest.mark.parametrize("lens,pre", [([300], [5000]), ([43, 900, 1], [70000, 0, 64]), ([1] * 80, [130] * 80),
                                      ([2000, 100], [1000, 40])])
def test_fixed_split_workspace_not_larger(hq, hkv, dqk, dv, lens, pre, splits):
    ws, info = _plan(hq, hkv, dqk, dv, lens, pre, splits)
    n = min(splits, max(1, max(pre) // 64))
    rows, bm = sum(lens), 256
    slots = sum((-(-x // bm) + 1) // 2 for x in lens)
    former = _a(2 * slots * n * 32) + (_a(n * rows * hq * dv * 4) + _a(n * rows * hq * 4) if n > 1 else 0)
    assert info.num_splits == n
    assert ws <= max(former, info.num_work_items * 32 + 256)
    assert info.num_work_items * 32 < (1 << 20)


@pytest.mark.parametrize("hq,hkv,dqk,dv,rows,pre", [
    (32, 8, 128, 128, 4096, 20480), (128, 128, 192, 128, 8192, 65536), (16, 16, 192, 128, 8192, 100000),
    (64, 4, 128, 128, 8192, 0), (64, 4, 128, 128, 8192, 60000), (32, 8, 128, 128, 3840, 30000),
])
def test_automatic_plans_of_equal_slots_fit(hq, hkv, dqk, dv, rows, pre):
    ws, _ = _plan(hq, hkv, dqk, dv, [rows], [pre], -1)
    assert ws <= B.NOALLOC_SCRATCH_BYTES
