"""The RGB stem convolution in strips of output rows: on small partitions a
block takes several rows, the last strip of an image is shorter, and several
rounds of strips run when the rows of one round exceed the LDS.  Against the
fp64 oracle; bar: one rounding to bf16 plus fp32 sums of at most 147 products
(infinity-norm relative error <= 2^-8)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, K, R, stride, pad, act, slots
    (1, 67, 48, 64, 7, 2, 3, 1, 1),    # 34 rows over 16 strips: 3 rows each, the last one 1
    (3, 61, 224, 64, 7, 2, 3, 1, 1),   # strips of the widest images
    (40, 20, 16, 64, 7, 2, 3, 0, 1),   # more images than blocks: one strip each
    (9, 224, 40, 32, 3, 2, 1, 2, 1),   # 112 rows in strips of 38
    (2, 37, 31, 64, 3, 1, 1, 1, 2),    # W % 8 != 0 in longer strips
    (5, 19, 24, 16, 3, 1, 0, 1, 1),    # no padding
    (2, 9, 9, 64, 7, 2, 6, 1, 3),      # padding almost as wide as the image
    (1, 3, 1, 16, 3, 1, 2, 0, 1),      # one column
]


@pytest.mark.parametrize("case", CASES, ids=["-".join(str(v) for v in c) for c in CASES])
def test_strips(oracle_mod, case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    N, H, W, K, R, st, pad, act, slots = case
    print("stem strips", case, flush=True)
    xb = inputs.normal_bf16(41, (N, H, W, 3))
    wb = inputs.normal_bf16(42, (K, R, R, 3), scale=(2.0 / (3 * R * R)) ** 0.5)
    w4 = np.zeros((K, R, R, 4), dtype=wb.dtype)
    w4[..., :3] = wb
    rng = np.random.default_rng(43)
    scale, shift = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.uniform(-0.2, 0.2, K).astype(np.float32)
    Ho, Wo = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    buf = gu.empty_bf16((N * Ho * Wo * K + 64,))
    buf.fill_(float("nan"))
    y = buf[:N * Ho * Wo * K].view(N, Ho, Wo, K)
    part = ds.Partition(slot_offset=0, n_slots=slots)
    dev = gu.dev_bf16(xb), gu.dev_bf16(w4), gu.dev_f32(scale), gu.dev_f32(shift)
    torch.cuda.synchronize()
    try:
        ds.conv2d_rgb(dev[0], dev[1], K, R, st, pad, dev[2], dev[3], act, y, stream=part.stream_ptr)
        part.synchronize()
    finally:
        part.destroy()
    got = gu.host(y)
    assert np.all(np.isfinite(got)) and bool(torch.isnan(buf[N * Ho * Wo * K:].float()).all())
    ref = oracle_mod.conv2d(oracle_mod.bf16_bits_to_f64(xb), oracle_mod.bf16_bits_to_f64(wb), st, pad) * scale + shift
    ref = np.clip(ref, 0 if act else -np.inf, 6 if act == 2 else np.inf)
    assert oracle_mod.rel_err(got, ref) <= 2.0 ** -8
