"""Plans that run_noalloc's 64 MiB scratch took stay within it (host only).

The former workspace: 32 bytes per entry of one-head tiles (128 or 256 rows) run in pairs, and
the fp32 partials of every row for a split count common to the chunk. Fixed counts: the
workspace must not exceed that. Automatic ones: chunks that the former rule kept within the
scratch must stay within it, whatever their pieces: many equal slots, mixes whose unbounded
plans would need more (with the former planner's own sizes), and many segments of which one is
cut into many pieces.
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
    assert ws <= former


@pytest.mark.parametrize("hq,hkv,dqk,dv,rows,pre", [
    (32, 8, 128, 128, 4096, 20480), (128, 128, 192, 128, 8192, 65536), (16, 16, 192, 128, 8192, 100000),
    (64, 4, 128, 128, 8192, 0), (64, 4, 128, 128, 8192, 60000), (32, 8, 128, 128, 3840, 30000),
])
def test_automatic_plans_of_equal_slots_fit(hq, hkv, dqk, dv, rows, pre):
    ws, _ = _plan(hq, hkv, dqk, dv, [rows], [pre], -1)
    assert ws <= B.NOALLOC_SCRATCH_BYTES


# (heads and dims, rows, prefixes, workspace of the former planner): chunks whose plans would need
# more than the scratch if nothing bounded their partials
FORMER = [
    ((224, 32, 192, 128), [51, 164, 297, 1, 1113], [2179, 229, 20496, 34255, 1794], 512),
    ((64, 4, 128, 128), [1562, 39, 155, 3], [26948, 0, 0, 0], 512),
    ((40, 8, 128, 128), [348], [105652], 43096832),
    ((128, 128, 192, 128), [323, 262, 324, 1693, 7, 3], [0, 80184, 67071, 519, 0, 112], 768),
    ((40, 8, 128, 128), [2620, 3, 451, 1669, 58], [96591, 989, 3814, 561, 1455], 1024),
    ((32, 8, 128, 128), [11, 197, 2, 14], [0, 28188, 0, 82376], 59183104),
    ((224, 32, 192, 128), [412, 835], [71455, 0], 256),
    ((24, 1, 128, 128), [36, 348], [158, 45044], 38044672),
    ((16, 16, 192, 128), [2183, 6], [74938, 0], 54218496),
    ((64, 4, 128, 128), [2, 1513, 13], [76490, 34980, 0], 512),
    ((128, 128, 192, 128), [2, 39, 75, 252, 822, 616], [0, 109529, 146, 125634, 0, 0], 512),
    ((16, 16, 192, 128), [864, 2], [47719, 1837], 57199104),
    ((64, 4, 128, 128), [351], [85566], 46365952),
    ((96, 4, 192, 128), [72, 962, 931, 12, 105, 41], [312, 23673, 0, 0, 80, 0], 512),
    ((24, 1, 128, 128), [1963, 13, 164, 8, 27], [6896, 12101, 11303, 0, 0], 53872128),
]


@pytest.mark.parametrize("heads,lens,pre,former", FORMER)
def test_automatic_mixes_stay_within_the_scratch(heads, lens, pre, former):
    assert former <= B.NOALLOC_SCRATCH_BYTES
    ws, _ = _plan(*heads, lens, pre, -1)
    assert ws <= B.NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("hq,hkv,nseg,prefix", [(64, 4, 65536, 1 << 20), (4, 1, 65536, 200000), (64, 4, 16384, 1 << 20)])
@pytest.mark.parametrize("others", [0, 700])
def test_many_segments_of_which_one_is_split(hq, hkv, nseg, prefix, others):
    """The former planner took 64 bytes a segment. A launch uses 60 (its table) and the split
    segment's partials; the listing of all (tile, piece) pairs is not part of it."""
    ws, info = _plan(hq, hkv, 128, 128, [1] * nseg, [prefix] + [others] * (nseg - 1), -1)
    partials = sum(_a(info.num_splits * hq * x * 4) for x in (128, 1)) if others == 0 else 1 << 20
    assert ws <= max(60 * nseg + 256 + partials, 1 << 20)


def test_partials_may_fill_the_scratch():
    """Only a launch table, past 64 segments, is taken off the room for partials: 3 pieces, which the
    former planner took here, need 61.3 MiB of the 64."""
    ws, info = _plan(12, 4, 64, 64, [6865], [96676], -1)
    assert info.num_splits == 3
    assert ws <= B.NOALLOC_SCRATCH_BYTES
