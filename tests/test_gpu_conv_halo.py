"""The 3x3 stride-1 kernel that keeps a tile's input pixels in LDS, on the GPU
against the fp64 oracle, and its dispatch rule on the host.

The cases sit where its tiles can go wrong: images narrower than a fragment
(1 pixel, 1 row, 1 column), tiles over several images, partial tiles of the
two-dimensional tiling at both edges, channel tails (K = 8, 72, 136), one and
several 64-channel chunks, every epilogue, a residual, a depth split, and a
launch in two parts (whole rounds of the large tile, then the rest).

Bar: one rounding to bf16 (2^-9 of a value) plus fp32 sums of at most 4608
bf16 products: infinity-norm relative error <= 2^-8."""
import numpy as np
import pytest

TOL = 2.0 ** -8

CASES = [
    # N, H, W, C, K, act, residual, n_cu
    (1, 1, 1, 64, 8, 1, False, 256),
    (3, 1, 9, 64, 72, 0, False, 64),
    (5, 9, 1, 128, 64, 2, True, 128),
    (2, 7, 7, 512, 136, 1, True, 64),      # tiles over both images
    (1, 7, 7, 512, 512, 1, False, 256),    # depth split
    (8, 14, 14, 320, 128, 3, False, 64),   # five chunks
    (9, 15, 16, 64, 128, 1, False, 64),    # BM + 2W + 2 rows still fit a patch
    (1, 37, 61, 128, 64, 4, False, 64),    # th x tw tiles, partial at both edges
    (1, 65, 33, 64, 128, 1, True, 64),
    (2, 56, 56, 128, 128, 1, False, 64),
    (8, 28, 28, 128, 256, 1, True, 64),    # 128 x 256 tiles
    (16, 28, 28, 128, 128, 0, False, 96),
]


def plan(ds, N, H, W, C, K, act, n_cu, **kw):
    return ds.conv2d_plan(N, H, W, C, K, 3, 3, 1, 1, act, False, n_cu, **kw)


def test_dispatch_rule():
    """Only 3x3, stride 1, pad 1, whole 64-channel chunks, K % 8 == 0, bf16
    output take the kernel, on fewer than 32 CUs only where the general plan does
    not split; its splits need the workspace."""
    import paper_2304_13541_amd as ds
    assert all(plan(ds, 16, 14, 14, 256, 256, 1, n)["kernel"] == 2 for n in (24, 32, 56, 128))
    assert plan(ds, 2, 9, 9, 256, 384, 1, 24)["kernel"] == 0 and plan(ds, 2, 9, 9, 256, 384, 1, 32)["kernel"] == 2
    for C, K, R, st, pad, f32, n_cu in [(256, 256, 3, 2, 1, False, 128), (256, 256, 3, 1, 0, False, 128),
                                        (256, 256, 5, 1, 2, False, 128), (256, 256, 1, 1, 0, False, 128),
                                        (264, 256, 3, 1, 1, False, 128), (256, 252, 3, 1, 1, False, 128),
                                        (256, 256, 3, 1, 1, True, 128)]:
        p = ds.conv2d_plan(16, 14, 14, C, K, R, R, st, pad, 1, f32, n_cu)
        assert p["kernel"] == 0, (C, K, R, st, pad, f32, n_cu, p)
    rng = np.random.default_rng(3)
    for _ in range(2000):
        N, H, W = (int(v) for v in rng.integers(1, [33, 120, 120]))
        C, K, n_cu = 64 * int(rng.integers(1, 9)), 8 * int(rng.integers(1, 65)), 8 * int(rng.integers(1, 33))
        p = plan(ds, N, H, W, C, K, 1, n_cu)
        assert p["workspace_bytes"] == (16384 + 4 * p["splits"] * N * H * W * K if p["splits"] > 1 else 0)
        assert p["kernel"] != 2 or p["workspace_bytes"] <= ds.conv2d_noalloc_scratch_bytes()
        assert p["tiles_per_split"] * p["splits"] >= 9 * C // 64 > p["tiles_per_split"] * (p["splits"] - 1)
        none = plan(ds, N, H, W, C, K, 1, n_cu, workspace_bytes=0)
        assert none["splits"] == 1 and none["workspace_bytes"] == 0


def test_tiles_and_splits():
    """The tiles that the kernel has, over the range of shapes; only 64 x 64 tiles split (a split 64 x 128 block needs
    the registers of a whole CU, which the estimate of two blocks per CU does not count)."""
    import paper_2304_13541_amd as ds
    rng = np.random.default_rng(5)
    seen = set()
    for _ in range(4000):
        N, H, W = (max(1, int(v)) for v in np.exp(rng.uniform(0, np.log([32, 112, 112]))))
        C, K, n_cu = 64 * int(rng.integers(1, 13)), 8 * int(rng.integers(1, 97)), 8 * int(rng.integers(1, 33))
        p = plan(ds, N, H, W, C, K, 1, n_cu)
        if p["kernel"] == 2:
            seen.add((p["tile_n"], p["tile_m"], p["splits"] > 1))
    assert seen == {(64, 128, False), (64, 64, False), (64, 64, True), (128, 256, False)}


@pytest.fixture(scope="module")
def env(oracle_mod):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    return ds, gu, inputs, oracle_mod, torch


def run(env, case, offset=0):
    """Outputs with the depth split and without, items checked, and the oracle's; `offset` shifts y by
    that many elements."""
    ds, gu, inputs, oracle, torch = env
    N, H, W, C, K, act, use_res, n_cu = case
    xb = np.maximum(inputs.normal_bf16(7, (N, H, W, C)).view(np.int16), 0).view(np.uint16)  # after a ReLU
    wb = inputs.normal_bf16(8, (K, 3, 3, C), scale=(2.0 / (9 * C)) ** 0.5)
    rng = np.random.default_rng(9)
    scale, shift = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.uniform(-0.2, 0.2, K).astype(np.float32)
    resb = inputs.normal_bf16(10, (N, H, W, K)) if use_res else None
    p = plan(ds, N, H, W, C, K, act, n_cu)
    ws = torch.zeros(max(p["workspace_bytes"], 16384) // 4, dtype=torch.int32, device="cuda:0")
    args = (gu.dev_bf16(xb), gu.dev_bf16(wb), K, 3, 3, 1, 1, gu.dev_f32(scale), gu.dev_f32(shift),
            gu.dev_bf16(resb) if use_res else None, act)
    got = []
    for w in (ws, None):
        buf = gu.empty_bf16((N * H * W * K + 8,))
        buf.fill_(float("nan"))
        y = buf[offset:offset + N * H * W * K].view(N, H, W, K)
        ds.conv2d_ws(*args, y, w, n_cu=n_cu)
        torch.cuda.synchronize()
        got.append(gu.host(y))
        assert bool(torch.isnan(buf[:offset].float()).all()) and bool(torch.isnan(buf[offset + y.numel():].float()).all())
    assert int(ws[:4096].abs().sum().item()) == 0, "split-K arrival counters must be back at zero"
    items = sorted({0, N // 2, N - 1})
    ref = oracle.conv2d(oracle.bf16_bits_to_f64(xb[items]), oracle.bf16_bits_to_f64(wb), 1, 1) * scale + shift
    if use_res:
        ref = ref + oracle.bf16_bits_to_f64(resb[items])
    if act in (1, 2):
        ref = np.clip(ref, 0, 6 if act == 2 else np.inf)
    elif act == 3:
        from scipy.special import erf
        ref = 0.5 * ref * (1.0 + erf(ref / np.sqrt(2.0)))
    elif act == 4:
        ref = np.tanh(ref)
    return p, [g[items] for g in got], ref


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=["-".join(str(v) for v in c) for c in CASES])
def test_conv_halo(env, case):
    print("conv halo case", case, flush=True)
    p, got, ref = run(env, case)
    errs = [env[3].rel_err(g, ref) for g in got]
    print("  plan", p, "rel_err", errs, flush=True)
    assert p["kernel"] == 2
    assert all(np.all(np.isfinite(g)) for g in got) and max(errs) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2, 14, 14, 128, 64, 1, False, 128), (8, 28, 28, 128, 64, 1, True, 64),
                                  (8, 28, 28, 128, 256, 1, True, 64), (1, 7, 7, 512, 512, 1, False, 256)],
                         ids=["64x64", "64x128", "128x256", "split"])
def test_unaligned_output_runs_the_planned_kernel(env, case):
    """A y that is 8 or 2 bytes past an aligned address holds the bits of an aligned one, with the split and without
    (the general kernel sums in another order)."""
    p, want, ref = run(env, case)
    assert p["kernel"] == 2 and max(env[3].rel_err(g, ref) for g in want) <= TOL
    for offset in (4, 1):
        _, got, _ = run(env, case, offset=offset)
        assert all(np.array_equal(g, w) for g, w in zip(got, want)), offset


@pytest.mark.gpu
def test_two_part_launch(env):
    """More images than whole rounds of the large tile hold: the last ones run in the small tile (11 images are
    68 large tiles on 64 CUs; two rounds of them would lose to the small tile alone)."""
    case = (11, 28, 28, 128, 256, 1, True, 64)
    p, got, ref = run(env, case)
    assert (p["kernel"], p["tile_n"], p["tile_m"]) == (2, 128, 256)
    assert max(env[3].rel_err(g, ref) for g in got) <= TOL
