"""kv_append_paged over head counts and dims around the kernel's cases, bit for bit (GPU).

A token's granules (16 bytes) are or are not a multiple of a wave's 64; head dims of 8 (one
granule) and odd granule counts go through the division by multiplication; one case is past
the size from which loads and stores are non-temporal; strided inputs; padding slots.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("tokens,heads,dqk,dv,page", [
    (1, 1, 8, 8, 64),          # 2 granules a token
    (33, 3, 24, 40, 64),       # 24
    (257, 1, 128, 128, 64),    # 32: two tokens a wave
    (100, 2, 192, 128, 128),   # 80
    (65, 4, 64, 64, 64),       # 64: one token a wave
    (130, 8, 128, 128, 64),    # 256
    (77, 16, 192, 128, 64),    # 640
    (19, 5, 1024, 8, 64),      # 645
    (2000, 128, 192, 128, 128),  # 5120, 164 MB of new rows
])
@pytest.mark.parametrize("strided", [False, True])
def test_append_shapes(tokens, heads, dqk, dv, page, strided):
    from paper_2608_26523_amd.attention import kv_append_paged
    print("case:", tokens, heads, dqk, dv, page, strided, flush=True)
    npages = -(-tokens // page) + 2
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens + heads)

    def new(d):
        x = torch.randint(-32768, 32767, (tokens, heads, d + 8 * strided), generator=g, device=DEV, dtype=torch.int16)
        return x.view(torch.bfloat16)[..., :d]

    k_new, v_new = new(dqk), new(dv)
    slots = torch.randperm(npages * page, generator=g, device=DEV)[:tokens]
    slots[tokens // 2] = -1
    if tokens > 2:
        slots[1] = npages * page
    k = torch.full((npages, page, heads, dqk), 3.0, device=DEV, dtype=torch.bfloat16)
    v = torch.full((npages, page, heads, dv), 3.0, device=DEV, dtype=torch.bfloat16)
    want_k, want_v = k.clone(), v.clone()
    ok = (slots >= 0) & (slots < npages * page)
    want_k.view(-1, heads, dqk)[slots[ok]] = k_new[ok]
    want_v.view(-1, heads, dv)[slots[ok]] = v_new[ok]
    kv_append_paged(k_new, v_new, k, v, slots)
    torch.cuda.synchronize()
    assert torch.equal(k.view(torch.int16), want_k.view(torch.int16))
    assert torch.equal(v.view(torch.int16), want_v.view(torch.int16))
