"""Layer norm and embedding sum at the edges of the one-wave rows (16-byte
pieces: H a multiple of 8, aligned tensors) and of the block per row that
takes the others, against the fp64 oracle; bar: one rounding to bf16 plus fp32
sums of at most 2048 values (infinity-norm relative error <= 2^-8)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# rows, H, element offset of the bf16 tensors, gamma and beta given
CASES = [(5, 8, 0, True), (3, 512, 0, False), (2, 520, 0, True), (7, 1024, 0, True), (1, 1032, 0, True),
         (3, 2048, 0, False), (3, 2044, 0, True), (4, 768, 1, True), (4, 768, 4, False)]


@pytest.mark.parametrize("rows,H,offset,affine", CASES)
def test_rows(oracle_mod, rows, H, offset, affine):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    print("layer norm rows", rows, H, offset, affine, flush=True)
    rng = np.random.default_rng(61)

    def at_offset(bits):
        buf = gu.empty_bf16((bits.size + 8,))
        buf.fill_(float("nan"))
        t = buf[offset:offset + bits.size].view(*bits.shape)
        t.copy_(gu.dev_bf16(bits))
        return t

    g = rng.normal(1, 0.3, H).astype(np.float32) if affine else np.ones(H, np.float32)
    b = rng.normal(0, 0.3, H).astype(np.float32) if affine else np.zeros(H, np.float32)
    gd, bd = (gu.dev_f32(g), gu.dev_f32(b)) if affine else (None, None)
    g, b = g.astype(np.float64), b.astype(np.float64)
    buf = gu.empty_bf16((rows * H + 8,))
    buf.fill_(float("nan"))
    y = buf[offset:offset + rows * H].view(rows, H)

    xb = inputs.normal_bf16(62, (rows, H), scale=3.0)
    ds.layernorm(at_offset(xb), gd, bd, 1e-12, y)
    torch.cuda.synchronize()
    f64 = oracle_mod.bf16_bits_to_f64
    assert bool(torch.isnan(buf[offset + rows * H:].float()).all())
    assert oracle_mod.rel_err(gu.host(y), oracle_mod.layernorm(f64(xb), g, b, 1e-12)) <= 2.0 ** -8

    web, peb, teb = (inputs.normal_bf16(s, (n, H), scale=0.5) for s, n in ((63, 11), (64, 4), (65, 1)))
    ids = rng.integers(0, 11, rows).astype(np.int32)
    T = min(rows, 4)
    ds.embed_ln(torch.from_numpy(ids).to("cuda:0"), T, at_offset(web), at_offset(peb), at_offset(teb), gd, bd, 1e-12, y)
    torch.cuda.synchronize()
    e = f64(web)[ids] + f64(peb)[np.arange(rows) % T] + f64(teb)[0]
    assert oracle_mod.rel_err(gu.host(y), oracle_mod.layernorm(e, g, b, 1e-12)) <= 2.0 ** -8
