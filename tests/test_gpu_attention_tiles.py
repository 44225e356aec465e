"""Attention core at the edges of its 16-token tiles, unaligned tensors and
values that must not leak through masked keys, against the fp64 oracle; bar:
one rounding to bf16 plus the fp32 softmax (infinity-norm relative error <=
2^-8 + 2^-10)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [(2, t, 3, o) for t in (1, 2, 15, 16, 17, 31, 32, 33, 47, 48) for o in (0, 1)] + [(300, 20, 12, 0)]


@pytest.mark.parametrize("B,T,heads,offset", CASES)
def test_tiles(oracle_mod, B, T, heads, offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    print("attention tiles", B, T, heads, offset, flush=True)
    w = heads * 64
    qkvb = inputs.normal_bf16(51, (B, T, 3 * w))
    src = gu.empty_bf16((B * T * 3 * w + 8,))
    src.fill_(float("nan"))  # rows past the last sequence
    qkv = src[offset:offset + B * T * 3 * w].view(B, T, 3 * w)
    qkv.copy_(gu.dev_bf16(qkvb))
    buf = gu.empty_bf16((B * T * w + 8,))
    buf.fill_(float("nan"))
    out = buf[offset:offset + B * T * w].view(B, T, w)
    ds.attention(qkv, heads, out)
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf[offset + B * T * w:].float()).all())
    ref = oracle_mod.attention(oracle_mod.bf16_bits_to_f64(qkvb), heads)
    assert oracle_mod.rel_err(gu.host(out), ref) <= 2.0 ** -8 + 2.0 ** -10


def test_infinite_value_row():
    """An infinite value in the last token's v gives an infinite output (its
    weight is positive), not NaN from the masked rows of its tile."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    qkv = torch.zeros(1, 20, 192, device="cuda", dtype=torch.bfloat16)
    qkv[0, 19, 128] = float("inf")
    out = torch.zeros(1, 20, 64, device="cuda", dtype=torch.bfloat16)
    ds.attention(qkv, 1, out)
    torch.cuda.synchronize()
    assert bool(torch.isinf(out[0, :, 0]).all()) and bool((out[0, :, 1:] == 0).all())
