"""The LSTM recurrence in one launch (workgroups exchanging h through device
memory), on the GPU against the fp64 oracle (h rounded to bf16 where it
enters the recurrent product).

The cases sit at the edges of its plan: one item, a full and a just
overfull batch slice (16 / 17), ragged slices, one depth step (H = 32), idle
waves (H = 96), the widest rows (H = 2048), partitions that hold the rows in
8, 4 and 2 tiles per workgroup, and engines of unequal size (5 and 10 slots).
Also: NaN inputs stay in their item, a wait that gives up at once, replays of
a captured launch.

Bar: h is a bf16 rounding apart from the oracle's at each step (2^-9), fed
back through gates of slope <= 1: infinity-norm relative error <= 2^-7."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2.0 ** -7

CASES = [
    # T, B, I, H, slots (None: the default stream, the whole GPU)
    (4, 1, 8, 32, 1),
    (5, 16, 16, 96, 2),
    (9, 17, 24, 96, 4),
    (6, 5, 64, 256, 6),
    (50, 32, 40, 512, 8),
    (12, 31, 64, 1024, 10),
    (7, 3, 64, 1024, 5),
    (20, 32, 64, 1024, 16),
    (20, 16, 64, 1024, None),
    (4, 9, 32, 1056, None),
    (5, 16, 32, 2048, None),
]


@pytest.fixture(scope="module")
def env(oracle_mod):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2304_13541_amd as ds
    from tests import gpu_util as gu
    from tests import inputs
    return ds, gu, inputs, oracle_mod, torch


class Layer:
    def __init__(self, env, T, B, I, H, nan=()):
        ds, gu, inputs, oracle, torch = env
        self.env, self.shape = env, (T, B, I, H)
        a = 1.0 / np.sqrt(H)
        self.xb = inputs.normal_bf16(31, (T, B, I))
        for t, b in nan:
            self.xb[t, b, 0] = 0x7fc0
        self.wih, self.whh = inputs.uniform_bf16(32, (4 * H, I), -a, a), inputs.uniform_bf16(33, (4 * H, H), -a, a)
        self.bias = np.random.default_rng(34).uniform(-2 * a, 2 * a, 4 * H).astype(np.float32)
        self.dev = [gu.dev_bf16(self.xb), gu.dev_bf16(self.wih), gu.dev_bf16(self.whh), gu.dev_f32(self.bias)]
        self.hb, self.hf = gu.empty_bf16((T, B, H)), gu.empty_f32((T, B, H))
        self.ws = torch.full((ds.lstm_workspace_bytes(T, B, H),), 0xA5, dtype=torch.uint8, device="cuda:0")

    def run(self, stream=None, **kw):
        self.env[0].lstm_layer(*self.dev, self.hb, self.hf, self.ws, stream=stream, **kw)

    def result(self):
        self.env[4].cuda.synchronize()
        return self.env[1].host(self.hb), self.env[1].host(self.hf)

    def ref(self):
        o = self.env[3]
        H = self.shape[3]
        return o.lstm_layer(o.bf16_bits_to_f64(self.xb), o.bf16_bits_to_f64(self.wih), o.bf16_bits_to_f64(self.whh),
                            self.bias.astype(np.float64), np.zeros(4 * H), round_h=True)[0]


@pytest.mark.parametrize("case", CASES, ids=["-".join(str(v) for v in c) for c in CASES])
def test_lstm_sequence(env, case):
    T, B, I, H, slots = case
    print("lstm sequence", case, flush=True)
    layer = Layer(env, T, B, I, H)
    part = env[0].Partition(slot_offset=0, n_slots=slots) if slots else None
    try:
        layer.run(part.stream_ptr if part else None)
        hb, hf = layer.result()
    finally:
        if part:
            part.destroy()
    ref = layer.ref()
    errs = [env[3].rel_err(v, ref) for v in (hb, hf)]
    print("  rel_err", errs, flush=True)
    assert max(errs) <= TOL


def test_scattered_slots(env):
    """Slots of one shader engine and one of another: the plan counts what the smaller one holds."""
    layer = Layer(env, 6, 4, 32, 512)
    part = env[0].Partition(slot_mask=0x11111113)
    try:
        layer.run(part.stream_ptr)
        hb, hf = layer.result()
    finally:
        part.destroy()
    assert env[3].rel_err(hf, layer.ref()) <= TOL


def test_nan_stays_in_its_item(env):
    """A NaN input makes its item NaN from that step on and no other item, also across batch slices."""
    layer = Layer(env, 8, 20, 32, 256, nan=[(2, 3), (5, 18)])
    layer.run()
    hb, hf = layer.result()
    clean = Layer(env, 8, 20, 32, 256)
    ref = clean.ref()
    want = np.zeros((8, 20), bool)
    want[2:, 3] = want[5:, 18] = True
    for v in (hb, hf):
        assert np.array_equal(np.isnan(v).all(axis=2), want) and np.array_equal(np.isnan(v).any(axis=2), want)
        assert env[3].rel_err(v[~want], ref[~want]) <= TOL


def test_wait_that_gives_up(env):
    """With no time to wait, one workgroup computes the sequence alone; the workspace then serves the normal path."""
    layer = Layer(env, 6, 18, 32, 128)
    ref = layer.ref()
    for wait in (-1, None, -1, 5000):
        layer.hf.fill_(7.0)
        layer.run(wait_us=wait)
        hb, hf = layer.result()
        assert env[3].rel_err(hf, ref) <= TOL and env[3].rel_err(hb, ref) <= TOL


def test_replays_equal_eager(env):
    """A captured layer replayed among eager work, each replay against the eager result (the exchange is cleared by a
    kernel of the launch itself)."""
    torch = env[4]
    layer = Layer(env, 10, 17, 32, 256)
    layer.run()
    want = [v.copy() for v in layer.result()]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        layer.run(torch.cuda.current_stream())
    for k in range(4):
        layer.hf.fill_(float(k))
        layer.hb.zero_()
        layer.ws.fill_(k)
        g.replay()
        hb, hf = layer.result()
        assert np.array_equal(hb, want[0]) and np.array_equal(hf, want[1])


def test_cells_are_those_of_the_step_path(env):
    """Without a recurrent product there is no sum to order: the one launch (4 steps) and the step path (3 steps)
    give the same bits.  Gates over the sigmoids' and tanh's ranges, the tanh gates densest around 1/4."""
    ds, gu, inputs, oracle, torch = env
    B, I, H = 3, 8, 1024
    rng = np.random.default_rng(41)
    bias = rng.uniform(-6, 6, 4 * H).astype(np.float32)
    bias[2 * H:3 * H] = np.concatenate([rng.uniform(-4, 4, H // 2), rng.uniform(0.2, 0.35, H // 2)])
    bias[:H // 4] = bias[3 * H:3 * H + H // 4] = 30.0  # open input and output gates: h = tanh(c)
    x, wih, whh = (gu.dev_bf16(np.zeros(s, np.uint16)) for s in ((4, B, I), (4 * H, I), (4 * H, H)))
    out = []
    for T in (3, 4):
        hb, hf = gu.empty_bf16((T, B, H)), gu.empty_f32((T, B, H))
        ws = torch.empty(ds.lstm_workspace_bytes(T, B, H), dtype=torch.uint8, device="cuda:0")
        ds.lstm_layer(x[:T], wih, whh, gu.dev_f32(bias), hb, hf, ws)
        torch.cuda.synchronize()
        out.append(hf.cpu().numpy()[:3])
    diff = np.abs(out[0].view(np.int32).astype(np.int64) - out[1].view(np.int32))
    print("  differing values", int((diff > 0).sum()), "largest distance, ulp", int(diff.max()), flush=True)
    assert np.array_equal(out[0], out[1])
