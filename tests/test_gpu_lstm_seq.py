"""The LSTM recurrence in one launch (workgroups exchanging h through device
memory), on the GPU against the fp64 oracle (h rounded to bf16 where it
enters the recurrent product).

The cases sit at the edges of its plan: one item, a full and a just
overfull batch slice (16 / 17), ragged slices, one depth step (H = 32), idle
waves (H = 96), the widest rows (H = 2048), partitions that hold the rows in
8, 4 and 2 tiles per workgroup, and engines of unequal size (5 and 10 slots).
The plan and the control words show which path ran.
Also: NaN inputs stay in their item, a wait that gives up at once, layers that
share CUs, replays of a captured launch.

Bar: h is a bf16 rounding apart from the oracle's at each step (2^-9), fed
back through gates of slope <= 1: infinity-norm relative error <= 2^-7."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2.0 ** -7

CASES = [
    # T, B, I, H, slots (None: the default stream, the whole GPU), row tiles per workgroup
    (4, 1, 8, 32, 1, 2),
    (5, 16, 16, 96, 2, 2),
    (9, 17, 24, 96, 4, 2),
    (6, 5, 64, 256, 6, 2),
    (50, 32, 40, 512, 8, 4),
    (12, 31, 64, 1024, 10, 8),
    (7, 3, 64, 1024, 5, 8),
    (20, 32, 64, 1024, 16, 4),
    (20, 16, 64, 1024, None, 2),
    (4, 9, 32, 1056, None, 2),
    (5, 16, 32, 2048, None, 2),
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

    def control(self):
        """(a wait gave up, steps done of each workgroup's rows) from the workspace's control words: the last 2304
        bytes of the part that holds the exchange; (0, zeros) where the one launch went through by itself."""
        T, B, _, H = self.shape
        end = sum((n + 255) // 256 * 256 for n in (T * B * 16 * H, B * H * 4, 8 * H * H))
        w = self.ws[end - 2304:end].cpu().numpy().view(np.int32)
        return int(w[1]), w[64:320]

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
    T, B, I, H, slots, row_tiles = case
    print("lstm sequence", case, flush=True)
    assert env[0].lstm_plan(T, B, H, 8 * slots if slots else 256)[0] == row_tiles
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
    gave_up, done = layer.control()  # the one launch ran, and went through by itself
    assert gave_up == 0 and not done.any()


def test_scattered_slots(env):
    """Eight slots of one shader engine and one of another: the plan counts twice what the smaller one holds, 16
    workgroups, all of which run at once."""
    layer = Layer(env, 6, 4, 32, 512)
    mask = 0x11111113
    assert env[0].lstm_plan(6, 4, 512, 72, sum(0xff << 8 * j for j in range(32) if mask >> j & 1)) == (8, 16)
    part = env[0].Partition(slot_mask=mask)
    try:
        layer.run(part.stream_ptr)
        hb, hf = layer.result()
    finally:
        part.destroy()
    assert env[3].rel_err(hf, layer.ref()) <= TOL
    gave_up, done = layer.control()
    assert gave_up == 0 and not done.any()


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


@pytest.mark.parametrize("B,H,slots", [(18, 128, None), (32, 1024, 16), (5, 256, 2), (17, 96, 1), (9, 1056, None)])
def test_wait_that_gives_up(env, B, H, slots):
    """With no time to wait, the workgroups that run compute the sequence as shared work; the workspace then serves
    the normal path."""
    T = 6
    layer = Layer(env, T, B, 32, H)
    ref = layer.ref()
    blocks = env[0].lstm_plan(T, B, H, 8 * slots if slots else 256)[1]
    part = env[0].Partition(slot_offset=0, n_slots=slots) if slots else None
    try:
        for wait in (-1, None, -1, 5000):
            layer.hf.fill_(7.0)
            layer.run(part.stream_ptr if part else None, wait_us=wait)
            hb, hf = layer.result()
            assert env[3].rel_err(hf, ref) <= TOL and env[3].rel_err(hb, ref) <= TOL
            gave_up, done = layer.control()
            assert gave_up == (wait == -1) and np.all(done[blocks:] == 0)
            assert np.all(done[:blocks] == (T if wait == -1 else 0))
    finally:
        if part:
            part.destroy()


@pytest.mark.parametrize("offsets,wait", [((0, 8, 4), None), ((0, 0, 0), None), ((0, 8, 4), 50)])
def test_layers_that_share_cus(env, offsets, wait):
    """Three recurrences released at once on CUs that they share, so that each may hold a part of them: whichever wait
    gives up, the results hold, and the wait and the shared work take a few milliseconds (bar: 20; all the work on one
    CU takes over 50).  A kernel on the default stream, which the partitions' streams wait for, releases them."""
    torch, ds = env[4], env[0]
    layers = [Layer(env, 50, 32, 32, 1024) for _ in offsets]
    ref = layers[0].ref()
    big = torch.zeros(1 << 28, device="cuda:0")
    parts = [ds.Partition(slot_offset=o, n_slots=16) for o in offsets]
    try:
        streams = [torch.cuda.ExternalStream(p.stream_ptr) for p in parts]
        for rep in range(4):
            for layer in layers:
                layer.hf.fill_(7.0)
            torch.cuda.synchronize()
            start = torch.cuda.Event(enable_timing=True)
            ends = [torch.cuda.Event(enable_timing=True) for _ in parts]
            for _ in range(3):
                big.add_(1.0)
            start.record()
            for layer, p, s, e in zip(layers, parts, streams, ends):
                layer.run(p.stream_ptr, wait_us=wait)
                e.record(s)
            results = [layer.result() for layer in layers]
            ms = max(start.elapsed_time(e) for e in ends)
            state = [layer.control() for layer in layers]
            print("  released together:", offsets, wait, "%.2f ms," % ms, "gave up", [s[0] for s in state], flush=True)
            for (hb, hf), (gave_up, done) in zip(results, state):
                assert env[3].rel_err(hf, ref) <= TOL and env[3].rel_err(hb, ref) <= TOL
                assert np.all(done[:128] == (50 if gave_up else 0))
            assert rep == 0 or ms < 20.0
    finally:
        for p in parts:
            p.destroy()


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
