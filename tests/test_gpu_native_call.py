"""The native extension's calls against the wrapper's general path (GPU).

A call with plain tensors on the current stream goes through the extension; anything else
comes back from it before any device work and is done, or refused, in Python. For forms that
both take (contiguous and strided tensors, with and without lse, larger buffers, parameters)
the results must be the same bits; for forms that neither takes, the same exception.
"""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


class _General:
    """Stands in for the extension's caller: takes nothing."""

    def __getattr__(self, name):
        return lambda *a: -1


def _rand(*shape, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + sum(shape))
    return (torch.randn(*shape, generator=g, device=DEV) / 8).to(torch.bfloat16)


def _setup(entry):
    from paper_2608_26523_amd.attention import ChunkAttention
    hq, hkv, dqk, dv = (4, 4, 192, 128) if entry == "run_mla" else (4, 2, 128, 128)
    n, p, page = 70, 130, 64
    attn = ChunkAttention(hq, hkv, dqk, dv, max_chunk_tokens=n, max_kv_len=p + n)
    attn.plan([0, n], [0], [p])
    args = {"q": _rand(n, hq, dqk), "out": torch.zeros(n, hq, dv, device=DEV, dtype=torch.bfloat16),
            "lse": torch.zeros(hq, n, device=DEV)}
    if entry == "run_paged":
        table = torch.tensor([[3, 0, 2, 1]], dtype=torch.int32, device=DEV)
        args.update(k_pages=_rand(5, page, hkv, dqk), v_pages=_rand(5, page, hkv, dv, seed=1), block_table=table)
    elif entry == "run_mla":
        args.update(k_nope=_rand(p + n, hkv, 128), k_rope=_rand(p + n, 64), v_cache=_rand(p + n, hkv, dv, seed=1))
    else:
        args.update(k_cache=_rand(p + n, hkv, dqk), v_cache=_rand(p + n, hkv, dv, seed=1))
    return attn, args


def _call(attn, entry, args, native):
    old = attn._native
    if not native:
        attn._native = _General()
    try:
        out, lse = getattr(attn, entry)(**args)
        torch.cuda.synchronize()
        return out.clone(), None if lse is None else lse.clone()
    finally:
        attn._native = old


def _strided(t, pad=8):
    """The same values in a view whose rows are further apart."""
    big = torch.zeros(t.shape[:-1] + (t.shape[-1] + pad,), dtype=t.dtype, device=t.device)
    v = big[..., :t.shape[-1]]
    v.copy_(t)
    return v


ENTRIES = ["run", "run_noalloc", "run_mla", "run_paged"]


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("form", ["plain", "strided", "no_lse", "long_lse", "parameter", "more_rows", "inference"])
def test_native_equals_general(entry, form):
    attn, args = _setup(entry)
    ref = _call(attn, entry, args, native=False)
    assert float(ref[0].float().abs().max()) > 0
    if form == "strided":
        args = {k: _strided(t) if t.dtype == torch.bfloat16 else t for k, t in args.items()}
    elif form == "no_lse":
        args["lse"] = None
    elif form == "long_lse":
        args["lse"] = torch.zeros(4, 300, device=DEV)[:, 100:170]
    elif form == "parameter":
        args["q"] = torch.nn.Parameter(args["q"], requires_grad=False)
    elif form == "more_rows":
        args["q"] = torch.cat([args["q"], _rand(9, *args["q"].shape[1:])])
        args["out"] = torch.zeros((100,) + tuple(args["out"].shape[1:]), dtype=torch.bfloat16, device=DEV)
    elif form == "inference":
        with torch.inference_mode():
            args["q"] = args["q"].clone()
    if args["lse"] is not None:
        args["lse"].zero_()
    args["out"].zero_()
    taken = []
    real = attn._native

    class _Spy:
        def __getattr__(self, name):
            def f(*a):
                taken.append(getattr(real, name)(*a))
                return taken[-1]
            return f

    attn._native = _Spy()
    out, lse = getattr(attn, entry)(**args)
    attn._native = real
    torch.cuda.synchronize()
    assert taken == [0], "the extension did not take this form"
    n = ref[0].shape[0]
    assert torch.equal(out[:n], ref[0])
    assert lse is None or torch.equal(lse, ref[1])


BAD = {
    "dtype": lambda a: a.update(q=a["q"].half()),
    "cpu": lambda a: a.update(q=a["q"].cpu()),
    "heads": lambda a: a.update(q=a["q"][:, :2]),
    "few_rows": lambda a: a.update(q=a["q"][:20]),
    "transposed": lambda a: a.update(q=a["q"].transpose(1, 2).contiguous().transpose(1, 2)),
    "out_dtype": lambda a: a.update(out=a["out"].float()),
    "lse_shape": lambda a: a.update(lse=a["lse"][:, :5]),
    "lse_stride": lambda a: a.update(lse=a["lse"].T.contiguous().T),
    "misaligned": lambda a: a.update(q=torch.zeros(a["q"].numel() + 1, dtype=a["q"].dtype, device=DEV)[1:].view(a["q"].shape)),
}


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("bad", sorted(BAD))
def test_refusals_are_the_same(entry, bad):
    attn, args = _setup(entry)
    BAD[bad](args)
    got = []
    for native in (False, True):
        with pytest.raises(Exception) as e:
            _call(attn, entry, args, native)
        got.append((e.type, str(e.value)))
    assert got[0] == got[1]


def test_append_native_equals_general():
    from paper_2608_26523_amd import binding as B
    from paper_2608_26523_amd.attention import kv_append_paged
    k_new, v_new = _rand(50, 2, 192), _rand(50, 2, 128, seed=1)
    slots = torch.randperm(256, device=DEV)[:50]
    res = []
    for stream in (None, torch.cuda.current_stream()):  # None: the extension; a stream: the general path
        k, v = torch.zeros(4, 64, 2, 192, device=DEV, dtype=torch.bfloat16), torch.zeros(4, 64, 2, 128, device=DEV, dtype=torch.bfloat16)
        if stream is None:
            assert B.load_torch().append(k_new, v_new, k, v, slots) == 0
        else:
            kv_append_paged(k_new, v_new, k, v, slots, stream=stream)
        torch.cuda.synchronize()
        res.append((k, v))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    assert float(res[0][0].float().abs().max()) > 0
    with pytest.raises(ValueError):
        kv_append_paged(k_new, v_new[:10], k, v, slots)
    with pytest.raises(TypeError):
        kv_append_paged(k_new.float(), v_new, k, v, slots)


def test_side_stream_and_closed_plan():
    """The extension launches on the stream that is current at the call, and takes nothing once
    the plan is closed."""
    attn, args = _setup("run")
    ref = _call(attn, "run", args, native=False)
    side = torch.cuda.Stream()
    args["out"].zero_()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        attn.run(**args)
    assert not side.query(), "the call did not go to the side stream"
    side.synchronize()
    assert torch.equal(args["out"], ref[0])
    attn.close()
    with pytest.raises(RuntimeError):
        attn.run(**args)


def test_graph_replays_equal_eager():
    """A chunk captured without a warm-up call (its launch table is in the kernel arguments) and
    replayed on new contents of its buffers, a split plan's merge among it; eager work of the
    same plan between the replays."""
    from paper_2608_26523_amd.attention import ChunkAttention
    hq, hkv, d, p, n = 4, 2, 128, 4000, 30
    attn = ChunkAttention(hq, hkv, d, d, max_chunk_tokens=n, max_kv_len=p + n)
    assert attn.plan([0, n], [0], [p]).num_splits > 1
    q, k, v = _rand(n, hq, d), _rand(p + n, hkv, d, seed=1), _rand(p + n, hkv, d, seed=2)
    out, lse = torch.zeros(n, hq, d, device=DEV, dtype=torch.bfloat16), torch.zeros(hq, n, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        attn.run(q, k, v, out, lse)
    for i in range(4):
        q.copy_(_rand(n, hq, d, seed=10 + i))
        v.copy_(_rand(p + n, hkv, d, seed=20 + i))
        ref, ref_lse = attn.run(q, k, v, torch.empty_like(out), torch.empty_like(lse))
        torch.cuda.synchronize()
        out.zero_()
        lse.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse), "replay %d" % i
