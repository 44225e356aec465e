"""64 x 64 and 32 x 128 convolution tiles in two depth groups (grids of at most one block
per CU): odd and even numbers of depth tiles, a depth tail, every addressing
mode, residual, fp32 output and depth slices, against the fp64 oracle; bar:
one rounding to bf16 plus fp32 sums of at most 3072 products (infinity-norm
relative error <= 2^-8)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, C, K, R, stride, pad, act, residual, fp32 output, splits
    (1, 5, 4, 384, 64, 1, 1, 0, 0, False, False, 1),    # 6 tiles
    (1, 9, 8, 448, 132, 1, 1, 0, 1, True, False, 1),    # 7 tiles: the second group sits one out
    (2, 7, 7, 488, 96, 1, 1, 0, 3, True, False, 1),     # depth tail
    (3, 1, 20, 768, 768, 1, 1, 0, 4, False, True, 1),   # fp32 output
    (1, 9, 9, 512, 128, 1, 2, 0, 1, False, False, 1),   # strided
    (1, 9, 7, 64, 64, 3, 2, 1, 2, False, False, 1),     # one window position per tile: 9 tiles
    (2, 11, 13, 40, 100, 3, 2, 1, 1, False, False, 1),  # general addressing, 6 tiles
    (1, 1, 20, 3072, 768, 1, 1, 0, 0, True, False, 8),  # slices of 6 tiles
    (2, 21, 33, 136, 20, 3, 2, 1, 2, False, False, 1),  # 32 x 128 tiles
    (1, 13, 12, 832, 32, 1, 1, 0, 1, True, False, 1),
]


@pytest.mark.parametrize("case", CASES, ids=["-".join(str(int(v)) for v in c) for c in CASES])
def test_groups(oracle_mod, case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    N, H, W, C, K, R, st, pad, act, use_res, f32, splits = case
    print("conv groups", case, flush=True)
    plan = ds.conv2d_plan(N, H, W, C, K, R, R, st, pad, act, f32, 256)
    assert (plan["tile_n"], plan["splits"], plan["stages"]) == (64 if K > 32 else 32, splits, 8)
    f64 = oracle_mod.bf16_bits_to_f64
    xb, wb = inputs.normal_bf16(71, (N, H, W, C)), inputs.normal_bf16(72, (K, R, R, C), scale=(2.0 / (C * R * R)) ** 0.5)
    Ho, Wo = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    resb = inputs.normal_bf16(73, (N, Ho, Wo, K))
    rng = np.random.default_rng(74)
    scale, shift = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.uniform(-0.2, 0.2, K).astype(np.float32)
    y = gu.empty_f32((N, Ho, Wo, K)) if f32 else gu.empty_bf16((N, Ho, Wo, K))
    ws = torch.zeros(max(plan["workspace_bytes"], 16384) // 4 + 64, dtype=torch.int32, device="cuda:0")
    for _ in range(2):  # the second launch finds the counters as the first left them
        ds.conv2d_ws(gu.dev_bf16(xb), gu.dev_bf16(wb), K, R, R, st, pad, gu.dev_f32(scale), gu.dev_f32(shift),
                     gu.dev_bf16(resb) if use_res else None, act, y, ws, out_fp32=f32, n_cu=256)
    torch.cuda.synchronize()
    v = oracle_mod.conv2d(f64(xb), f64(wb), st, pad) * scale + shift + (f64(resb) if use_res else 0.0)
    if act in (1, 2):
        v = np.clip(v, 0.0, 6.0 if act == 2 else np.inf)
    elif act:
        t = torch.from_numpy(v)
        v = (torch.nn.functional.gelu(t) if act == 3 else torch.tanh(t)).numpy()
    assert oracle_mod.rel_err(gu.host(y), v) <= 2.0 ** -8
