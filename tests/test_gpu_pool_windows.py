"""Max pools with 2x2 and 3x3 windows (all loads in flight) and with other
windows (a loop), at padded and ragged edges, against the oracle; a max of
bf16 values is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 8, 3, 1, 1), (2, 5, 1, 24, 2, 1, 1), (3, 13, 17, 40, 3, 2, 1), (2, 9, 7, 16, 3, 3, 2),
         (1, 6, 5, 8, 2, 3, 0), (2, 11, 10, 16, 5, 2, 2), (1, 4, 4, 8, 1, 2, 0), (5, 112, 112, 64, 3, 2, 1)]


@pytest.mark.parametrize("case", CASES, ids=["-".join(str(v) for v in c) for c in CASES])
def test_windows(oracle_mod, case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    N, H, W, C, k, st, pad = case
    print("pool windows", case, flush=True)
    xb = inputs.normal_bf16(81, (N, H, W, C))
    n = N * ((H + 2 * pad - k) // st + 1) * ((W + 2 * pad - k) // st + 1) * C
    buf = gu.empty_bf16((n + 64,))
    buf.fill_(float("nan"))
    y = buf[:n].view(N, (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1, C)
    ds.maxpool(gu.dev_bf16(xb), k, st, pad, y)
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf[n:].float()).all())
    assert np.array_equal(gu.host(y), oracle_mod.maxpool(oracle_mod.bf16_bits_to_f64(xb), k, st, pad))
