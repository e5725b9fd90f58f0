"""The XCD-resident kernel at the sizes where its indexing and its exchange can go wrong, against the CPU oracle: every tile
height, first and last width of each, input widths around a wave's loads, 1, 2, 3 and 16 + 1 sequences, fewer and more steps than
a slot is marked ahead, both directions, several launches, several passes, the projection in front, padded widths in either
layout, and the GRU with the reset gate before the product in the same shapes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {0: 1e-4, 1: 2e-2}

SHAPES = [
    # cell, L, D, I, H, T, B, dtype
    (0, 1, 1, 128, 128, 1, 1, 1),       # one step: nothing is exchanged
    (0, 2, 1, 128, 128, 1, 3, 1),       # one step through two layers
    (1, 2, 1, 40, 128, 2, 2, 1),        # input of one and a quarter K blocks, rows read without the turn through LDS
    (0, 3, 1, 136, 256, 5, 17, 1),      # a second block of one sequence; as many steps as a slot is marked ahead, and one
    (1, 2, 1, 1024, 384, 9, 3, 1),      # widest input inside, three chunks per wave
    (0, 2, 1, 1032, 256, 6, 5, 1),      # wider than that: projection, layers above fused
    (0, 2, 2, 384, 384, 10, 33, 1),     # both directions, the second launch reads the first one's chunks (six loads per wave)
    (0, 5, 1, 512, 512, 13, 40, 1),     # more groups than XCDs: two launches
    (1, 2, 1, 512, 512, 7, 150, 1),     # one layer per launch, or several passes
    (0, 2, 2, 200, 200, 8, 20, 1),      # padded to 256 units
    (0, 2, 1, 56, 520, 6, 4, 1),        # (padded to 640 units: beyond this kernel)
    (0, 1, 1, 12, 32, 7, 4, 0),         # fp32 narrower than a wave's load
    (1, 3, 1, 20, 64, 11, 3, 0),
    (0, 2, 1, 7, 64, 6, 2, 0),          # fp32 input rows that are not whole chunks: projection
    (0, 12, 1, 64, 64, 20, 8, 0),       # twelve layers, two groups per XCD
    (0, 2, 2, 128, 128, 9, 18, 0),
    (0, 1, 1, 500, 256, 6, 16, 0),
    (0, 2, 1, 512, 512, 6, 1, 0),       # (tagged words)
    (0, 2, 1, 512, 512, 6, 2, 0),
    (0, 2, 1, 512, 512, 6, 70, 0),      # the longest products; a last block of six sequences
    (0, 1, 1, 512, 512, 4, 520, 1),     # passes of another kernel, the last eight sequences on this one
    (0, 1, 1, 64, 504, 3, 520, 1),      # the same through copies at the padded width
    (0, 1, 1, 512, 512, 4, 129, 0),     # passes of 128 sequences; the last one, alone, would run on tagged words
    (0, 2, 2, 300, 300, 4, 65, 0),      # the same padded, both directions, two launches
    (0, 1, 1, 20, 512, 4, 150, 0),      # passes of 128 and 22 behind one projection (input narrower than an eighth of the layer)
    (0, 2, 2, 520, 512, 3, 70, 0),      # ... (wider than the x waves hold), both directions; the second layer projects by itself
    (1, 2, 1, 504, 64, 7, 5, 1),        # inputs of four chunks a wave (with the reset gate before the product a step ahead still)
    (1, 2, 1, 520, 128, 8, 18, 1),      # ... of more (then in the step itself)
    (1, 2, 1, 248, 64, 7, 9, 0),        # the same line in fp32
    (1, 1, 1, 260, 128, 5, 40, 0),
    (1, 1, 1, 40, 512, 4, 150, 1),      # one pass of another kernel; with the reset gate before the product, as above
    (0, 4, 1, 1024, 1024, 1, 5, 1),     # groups on two XCDs: one step, the whole chip
    (0, 4, 1, 1024, 1024, 11, 12, 1),   # chunk rows wider than the batch
    (0, 2, 1, 128, 128, 24, 3, 1),      # too few steps for the upper layer to run its input product a step ahead
    (1, 2, 1, 512, 512, 25, 9, 1),      # just enough, an odd number
    (0, 3, 1, 64, 64, 50, 5, 0),
    (0, 2, 2, 512, 512, 6, 72, 1),      # passes of 64 and 8 sequences where a launch of larger tiles holds all 72
    (1, 3, 2, 40, 200, 5, 140, 1),      # the same padded, 128 and 12, a narrow input inside
    (0, 4, 1, 520, 256, 6, 300, 1),     # 256 and 44, the last pass with all layers in a launch
    (0, 2, 1, 1024, 1024, 6, 4, 1),     # (few steps of few sequences: tagged words)
    (0, 2, 1, 1024, 1024, 8, 4, 1),     # (as many as this kernel takes)
    (0, 4, 1, 768, 768, 24, 1, 1),      # one sequence, several layers in a launch
    (1, 1, 1, 640, 640, 12, 1, 1),      # ... one layer
    (0, 2, 2, 80, 640, 9, 3, 1),        # both directions, the second layer behind a projection
    (0, 2, 1, 1024, 1024, 12, 258, 1),  # a last pass of two sequences
    (0, 2, 1, 768, 768, 24, 64, 1),     # a launch for each layer where large tiles hold both in one
    (1, 4, 1, 1024, 1024, 9, 20, 1),    # two launches of two layers
    (0, 1, 1, 80, 640, 50, 100, 1),     # passes of 64 and 36 sequences
    (0, 2, 2, 80, 1000, 20, 44, 1),     # padded, passes of 32 and 12, the second layer behind a projection
    (1, 1, 1, 1032, 1024, 6, 40, 1),    # projection in front, three blocks of sequences
    (0, 2, 1, 40, 600, 9, 17, 1),       # padded to 640 units: 20 workgroups on either XCD
    (1, 2, 2, 768, 768, 7, 20, 1),      # both directions, the second launch behind a projection
    (0, 1, 1, 896, 896, 6, 5, 1),       # padded to 1024
    (0, 2, 1, 1280, 1280, 6, 9, 1),     # groups on all XCDs: 160 workgroups, the second layer reads the first one's chunks
    (1, 2, 1, 40, 1536, 7, 16, 1),      # 192, a narrow input
    (0, 1, 1, 1032, 1400, 5, 3, 1),     # padded, an input of nine loads a wave
    (0, 2, 1, 2048, 2048, 6, 16, 1),    # every compute unit, the state in two halves
    (1, 1, 1, 64, 2048, 1, 2, 1),       # one step of it
    (0, 1, 1, 2056, 1800, 9, 20, 1),    # two passes behind a projection
    (0, 1, 1, 1536, 1536, 33, 6, 1),    # many more steps than a slot is marked ahead
    (1, 1, 1, 64, 2048, 26, 3, 1),
    (0, 2, 1, 1032, 768, 9, 8, 1),      # several layers behind a projection, six chunk loads a wave: a loop of one load
    (1, 3, 1, 40, 384, 7, 17, 1),       # ... three
    (0, 2, 1, 80, 1024, 6, 16, 1),      # ... eight
    (0, 3, 1, 640, 640, 24, 1, 1),      # few sequences: eight K blocks a load, of five
    (1, 4, 1, 640, 640, 10, 3, 1),      # ... four, a load of one behind it
    (0, 2, 1, 768, 768, 9, 7, 1),       # ... two
    (0, 1, 1, 1280, 1280, 6, 2, 1),     # ... eight, of ten
    (1, 1, 1, 64, 1536, 9, 8, 1),       # ... two
    (0, 1, 1, 2048, 2048, 6, 8, 1),
    (0, 1, 1, 2048, 2048, 5, 4, 1),
    (0, 2, 1, 2048, 2048, 9, 7, 1),     # ... one, on rows as wide; two in the layer above
    (1, 1, 1, 80, 2048, 6, 5, 1),       # ... two
    (0, 1, 2, 64, 384, 15, 18, 1),      # one step fewer than the slots of a sequence that are used in turn,
    (1, 2, 1, 400, 400, 16, 9, 1),      # as many,
    (0, 1, 1, 128, 512, 17, 20, 1),     # one more,
    (1, 1, 2, 64, 128, 65, 17, 0),      # four times as many and one, fp32
    (0, 1, 1, 64, 128, 17, 3, 0),
    (1, 2, 1, 128, 256, 64, 5, 1),      # narrower layers: four times as many,
    (0, 2, 1, 128, 128, 16, 9, 1),      # as many,
    (1, 3, 1, 40, 256, 33, 2, 1),       # twice as many and one
]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_11339_amd import harness, rnn, workloads
    rnn.load_library()
    return harness, rnn, workloads


def _workload(W, shape, ragged):
    cell, L, D, I, H, T, B, dtype = shape
    cfg = W.Config("xcd", cell, L=L, D=D, I=I, H=H, T=T, B=B, dtype=dtype, seed=W.BASE_SEED + 3000 + H + 7 * B + T,
                   h0_std=0.5, len_min=1 if ragged else None)
    wl = W.make_workload(cfg, zero_pad_x=False)
    if cell == 0:
        wl.c0 = np.random.default_rng(cfg.seed).uniform(-1, 1, size=(L * D, B, H)).astype(np.float32)
    return wl


def _check(harness, wl, io, ref):
    y, hT, cT, ybits = harness.results(io)
    tol = TOL[wl.cfg.dtype]
    assert np.abs(y - ref[0]).max() <= tol and np.abs(hT - ref[1]).max() <= tol
    if wl.cfg.cell == 0:
        assert np.abs(cT - ref[2]).max() <= tol
    if wl.lengths is not None:
        for j, n in enumerate(wl.lengths):
            assert np.all(ybits[int(n):, j] == 0), "padded positions must be +0.0 bit patterns"


@pytest.mark.parametrize("ragged", [False, True], ids=["full", "ragged"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[:7] + ("f32" if s[7] == 0 else "bf16",)))
def test_against_oracle(gpu, oracle, shape, ragged):
    """Three calls (the second and third on memory the first left behind) agree bit for bit, and with the oracle; so does
    the batch-first call."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, ragged)
    c = wl.cfg
    print("\n  case %r ragged %r" % (shape, ragged), flush=True)
    model = harness.DeviceModel(wl)
    io = harness.DeviceIO(wl)
    harness.forward(model, io)
    _check(harness, wl, io, oracle.forward_workload(wl, nthreads=8))
    y, hT = io.y.clone(), io.hT.clone()
    for _ in range(2):
        io.y.fill_(7.0)
        harness.forward(model, io)
        torch.cuda.synchronize()
        assert torch.equal(io.y, y) and torch.equal(io.hT, hT)
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    assert rnn.rnn_model_set_batch_first(model.handle, 1) == rnn.RNN_OK
    y_bf = torch.full((c.B, c.T, c.D * c.H), 7.0, dtype=io.y.dtype, device="cuda")
    assert rnn.rnn_forward(model.handle, io.x.transpose(0, 1).contiguous(), io.lengths, io.h0, io.c0, y_bf, io.hT, io.cT, c.T, c.B,
                           torch.cuda.current_stream()) == rnn.RNN_OK
    torch.cuda.synchronize()
    assert torch.equal(y_bf.transpose(0, 1), y) and torch.equal(io.hT, hT)
    model.close()


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == 1] + [(1, 1, 2, 64, 256, 1, 5, 1)],
                         ids=lambda s: "L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[1:7] + ("f32" if s[7] == 0 else "bf16",)))
def test_reset_gate_before_the_product(gpu, oracle, shape):
    harness, rnn, W = gpu
    wl = _workload(W, shape, True)
    print("\n  case %r" % (shape,), flush=True)
    model = harness.DeviceModel(wl)
    assert rnn.rnn_model_set_gru_reset_before(model.handle, 1) == rnn.RNN_OK
    io = harness.DeviceIO(wl)
    harness.forward(model, io)
    _check(harness, wl, io, oracle.forward_workload(wl, nthreads=8, gru_variant=1))
    assert rnn.rnn_model_set_clip(model.handle, 0.4) == rnn.RNN_OK
    harness.forward(model, io)
    _check(harness, wl, io, oracle.forward_workload(wl, nthreads=8, gru_variant=1, clip=0.4))
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    model.close()


@pytest.mark.parametrize("shape", [
    (0, 2, 1, 512, 512, 800, 17, 1, 0, 0),      # slots in turn: two blocks of 16 take 75 MiB, tagged words 54
    (0, 2, 1, 1024, 1024, 400, 17, 1, 0, 0),    # the same on two XCDs
    (1, 4, 2, 384, 384, 461, 17, 1, 1, 0),      # both directions, batch-first
    (1, 6, 1, 8, 360, 323, 12, 1, 0, 1),        # r * h in turn as well
    (1, 16, 1, 48, 148, 358, 22, 0, 1, 1),      # ... and four layers to a launch instead of eight
    (0, 4, 2, 12, 512, 20, 374, 0, 0, 0),       # passes that project their own sequences
    (0, 4, 2, 12, 512, 14, 374, 0, 1, 0),
    (1, 4, 1, 1712, 512, 286, 22, 1, 0, 1),     # left to the cellwise plan
    (0, 1, 1, 1608, 1536, 110, 24, 1, 0, 0),    # on all eight XCDs, passes that project their own sequences
], ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s_bf%d_rb%d" % (s[:7] + ("f32" if s[7] == 0 else "bf16",) + s[8:]))
def test_static_array_that_only_tagged_words_fit(gpu, shape):
    """Calls whose workspace with a slot for every step exceeds the static array of 64 MiB, and that fit without this kernel: the
    bits of rnn_forward all the same (of the cellwise plan where only that one fits)."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape[:8], True)
    c = wl.cfg
    print("\n  case %r" % (shape,), flush=True)
    model, io, io2 = harness.DeviceModel(wl), harness.DeviceIO(wl), harness.DeviceIO(wl)
    if shape[9]:
        assert rnn.rnn_model_set_gru_reset_before(model.handle, 1) == rnn.RNN_OK
    if shape[3] == 1712:
        assert rnn.rnn_model_set_plan(model.handle, rnn.RNN_PLAN_CELLWISE) == rnn.RNN_OK
    assert rnn.rnn_model_set_batch_first(model.handle, shape[8]) == rnn.RNN_OK
    stream = torch.cuda.current_stream()
    if shape[8]:
        for t in (io, io2):
            t.x, t.y = t.x.transpose(0, 1).contiguous(), t.y.view(c.B, c.T, c.D * c.H)
    assert rnn.rnn_forward(model.handle, io.x, io.lengths, io.h0, io.c0, io.y, io.hT, io.cT, c.T, c.B, stream) == rnn.RNN_OK
    assert rnn.rnn_model_set_plan(model.handle, rnn.RNN_PLAN_AUTO) == rnn.RNN_OK
    for _ in range(2):
        assert rnn.rnn_forward_static(model.handle, io2.x, io2.lengths, io2.h0, io2.c0, io2.y, io2.hT, io2.cT, c.T, c.B,
                                      stream) == rnn.RNN_OK
        torch.cuda.synchronize()
        assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
        assert torch.equal(io.y, io2.y) and torch.equal(io.hT, io2.hT)
        assert c.cell == 1 or torch.equal(io.cT, io2.cT)
        io2.y.fill_(7.0)
    model.close()


@pytest.mark.parametrize("shape", [(0, 1, 1, 128, 128, 1, 1, 1), (0, 4, 1, 512, 512, 1, 16, 1), (1, 2, 1, 64, 200, 1, 17, 1),
                                   (0, 2, 1, 256, 256, 1, 40, 0), (0, 2, 2, 384, 384, 1, 5, 1), (0, 2, 1, 1024, 1024, 1, 8, 1),
                                   (0, 4, 1, 1024, 1024, 1, 1, 1), (1, 1, 1, 512, 512, 1, 300, 1), (0, 1, 1, 40, 1280, 1, 3, 1),
                                   (1, 2, 1, 1536, 1536, 1, 16, 1), (0, 2, 1, 2048, 2048, 1, 9, 1)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[:7] + ("f32" if s[7] == 0 else "bf16",)))
def test_state_of_a_stream_in_place(gpu, shape):
    """One frame per call, the state updated in place (hT = h0, cT = c0): every workgroup of a layer reads the h0 of all units, and
    none may write its hT before all have.  Bit for bit the stream with the two states in buffers of their own."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg
    print("\n  case %r" % (shape,), flush=True)
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    x = torch.randn((20,) + tuple(io.x.shape), device="cuda", generator=torch.Generator("cuda").manual_seed(c.seed % 1000)).to(io.x.dtype)
    c0 = io.c0 if io.c0 is not None else torch.zeros_like(io.h0)
    stream = torch.cuda.current_stream()

    def run(in_place):
        h, cc, ys = io.h0.clone(), c0.clone(), []
        for k in range(x.shape[0]):
            hn, cn = (h, cc) if in_place else (torch.full_like(h, 7.0), torch.full_like(cc, 7.0))
            assert rnn.rnn_forward(model.handle, x[k], None, h, cc, io.y, hn, cn, 1, c.B, stream) == rnn.RNN_OK
            ys.append(io.y.clone())
            h, cc = hn, (cn if c.cell == 0 else cc)
        torch.cuda.synchronize()
        assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
        return torch.stack(ys), h, cc

    want = run(False)
    for _ in range(3):
        for a, b in zip(run(True), want):
            assert torch.equal(a, b)
    model.close()


def test_rows_of_x_more_than_4_gib_apart(gpu):
    """A batch-first x of 16 sequences of 140000 steps of 1024 features: sequences 14 and 15 begin beyond 2^32 bytes.  Bit for bit
    the time-major call, whose rows of a step lie side by side."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, (0, 1, 1, 1024, 128, 2, 16, 1), False)
    model, T, B = harness.DeviceModel(wl), 140000, 16
    x = torch.randn((T, B, 1024), dtype=torch.bfloat16, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    y = [torch.full((T, B, 128), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    stream = torch.cuda.current_stream()
    assert rnn.rnn_forward(model.handle, x, None, None, None, y[0], None, None, T, B, stream) == rnn.RNN_OK
    assert rnn.rnn_model_set_batch_first(model.handle, 1) == rnn.RNN_OK
    x_bf, y_bf = x.transpose(0, 1).contiguous(), y[1].view(B, T, 128)
    assert rnn.rnn_forward(model.handle, x_bf, None, None, None, y_bf, None, None, T, B, stream) == rnn.RNN_OK
    torch.cuda.synchronize()
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    for b in range(B):
        assert torch.equal(y_bf[b], y[0][:, b]), b
    model.close()


@pytest.mark.parametrize("shape", [(0, 1, 1, 80, 256, 5, 4, 1), (0, 2, 1, 40, 128, 4, 2, 1), (0, 1, 2, 136, 384, 4, 17, 1),
                                   (0, 1, 1, 20, 64, 5, 3, 0), (0, 1, 1, 80, 768, 4, 16, 1), (0, 2, 1, 1024, 128, 4, 5, 1),
                                   (0, 1, 1, 80, 1536, 4, 16, 1), (0, 1, 1, 1032, 1536, 4, 5, 1)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[:7] + ("f32" if s[7] == 0 else "bf16",)))
def test_an_infinite_feature_saturates_the_gates(gpu, oracle, shape):
    """One infinite feature among the first of a row: every weight of it is finite and not zero, so the gates saturate and all
    results are finite.  Lanes whose chunk lies beyond the input must not make it zero times infinity."""
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg
    for w in wl.weights:
        w[w == 0.0] = 0.125
    wl.x[0, 0, 1] = np.inf
    wl.x[c.T - 1, c.B - 1, 0] = -np.inf
    print("\n  case %r" % (shape,), flush=True)
    ref = oracle.forward_workload(wl, nthreads=8)
    assert np.isfinite(ref[0]).all() and np.isfinite(ref[2]).all()
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    harness.forward(model, io)
    _check(harness, wl, io, ref)
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    model.close()


@pytest.mark.parametrize("shape", [(0, 2, 1, 128, 128, 9, 3, 1), (1, 3, 1, 256, 256, 12, 17, 1), (0, 2, 1, 512, 512, 14, 16, 1),
                                   (0, 2, 2, 384, 384, 10, 33, 1), (0, 12, 1, 64, 64, 20, 8, 0), (1, 1, 1, 256, 256, 9, 5, 0),
                                   (0, 2, 1, 512, 512, 8, 20, 0),
                                   # state slots in turn: written, read and marked again several times over
                                   (0, 2, 1, 512, 512, 40, 9, 1), (1, 2, 1, 128, 128, 80, 5, 1), (1, 1, 1, 256, 256, 80, 18, 0)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[:7] + ("f32" if s[7] == 0 else "bf16",)))
@pytest.mark.parametrize("reset_before", [0, 1])
def test_a_group_that_is_not_on_one_xcd(gpu, shape, reset_before):
    """The exchange through memory, which a group uses that the dispatcher has laid over several XCDs: the same bits."""
    import torch
    harness, rnn, W = gpu
    if reset_before and shape[0] == 0:
        shape = (1,) + shape[1:]
    wl = _workload(W, shape, True)
    print("\n  case %r reset before %d" % (shape, reset_before), flush=True)
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    assert rnn.rnn_model_set_gru_reset_before(model.handle, reset_before) == rnn.RNN_OK
    harness.forward(model, io)
    torch.cuda.synchronize()
    want = (io.y.clone(), io.hT.clone(), io.cT.clone())
    assert rnn.rnn_model_set_device_scope(model.handle, 2) == rnn.RNN_EINVAL
    assert rnn.rnn_model_set_device_scope(model.handle, 1) == rnn.RNN_OK
    for _ in range(3):
        io.y.fill_(7.0)
        harness.forward(model, io)
        torch.cuda.synchronize()
        assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
        assert torch.equal(io.y, want[0]) and torch.equal(io.hT, want[1]) and (shape[0] == 1 or torch.equal(io.cT, want[2]))
    model.close()


@pytest.mark.parametrize("shape,bound", [((0, 2, 1, 512, 512, 40, 32, 0), 4.1e-7), ((0, 1, 2, 64, 128, 64, 33, 0), 2.93e-7)],
                         ids=["two_layers_512", "both_directions_128"])
def test_fp32_sums_of_the_two_products_are_kept_apart(gpu, oracle, shape, bound):
    """Distance of the fp32 state from the 64-bit oracle (2-norm over 2-norm).  Products of the input and of the state in chains of
    their own: 3.63e-7 and 2.77e-7 (as on the tag-in-data kernel, 3.64e-7 and 2.77e-7; weights uniform in 1 / sqrt(H), x normal);
    in one chain 4.67e-7 and 3.09e-7.  The bound is the middle; over seeds the distances vary by less than 2 %."""
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg
    rng = np.random.default_rng(11)
    wl.weights = [rng.uniform(-c.H ** -0.5, c.H ** -0.5, size=w.shape).astype(np.float32) for w in wl.weights]
    wl.x = rng.standard_normal(wl.x.shape).astype(np.float32)
    wl.h0, wl.c0 = np.zeros_like(wl.h0), np.zeros_like(wl.h0)
    ref = oracle.forward_workload(wl, nthreads=8)
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    harness.forward(model, io)
    _, hT, _, _ = harness.results(io)
    rel = float(np.linalg.norm(hT - ref[1]) / np.linalg.norm(ref[1]))
    print("\n  case %r: hT %.3e" % (shape, rel), flush=True)
    assert rel <= bound
    model.close()


@pytest.mark.parametrize("shape,bound", [((0, 1, 1, 1536, 1536, 4, 8, 1), 1.63e-7), ((0, 1, 1, 2048, 2048, 4, 5, 1), 1.8e-7),
                                         ((0, 1, 2, 512, 512, 48, 72, 1), 1.24e-7), ((0, 1, 2, 256, 256, 48, 136, 1), 1.13e-7),
                                         ((0, 1, 1, 1024, 1024, 4, 8, 1), 1.45e-7), ((0, 1, 1, 768, 768, 4, 16, 1), 1.35e-7)],
                         ids=["1536_units", "2048_units", "passes_of_512_units", "passes_of_256_units", "1024_units", "768_units"])
def test_bf16_sums_of_the_two_products_are_kept_apart(gpu, shape, bound):
    """Distance of cT after one step from 64 bits (2-norm over 2-norm; the cell state is not rounded to bf16, so it shows the sums).
    Products of the input and of the state in chains of their own: 1.35e-7, 1.45e-7, 1.13e-7 and 1.08e-7 (the kernels that ran these
    shapes before 1.37e-7, 1.46e-7, 1.29e-7 and 1.14e-7); in one chain 1.92e-7, 2.17e-7, 1.35e-7 and 1.18e-7.  1024 and 768 units:
    1.26e-7 and 1.20e-7, in one chain 1.65e-7 and 1.50e-7.  The bound is the middle."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, True)
    c = wl.cfg
    rng = np.random.default_rng(11)
    bf16 = lambda a: W.bf16_bits_to_f32(W.f32_to_bf16_bits(a.astype(np.float32))).reshape(a.shape)
    wl.weights = [bf16(rng.uniform(-c.H ** -0.5, c.H ** -0.5, size=w.shape)) for w in wl.weights]
    wl.x, wl.h0 = bf16(rng.standard_normal(wl.x.shape)), bf16(0.3 * rng.standard_normal(wl.h0.shape))
    wl.c0 = (0.3 * rng.standard_normal(wl.h0.shape)).astype(np.float32)
    wl.lengths = np.ones(c.B, dtype=np.int32)
    want = []
    for d in range(c.D):
        w_ih, w_hh, b_ih, b_hh = [torch.from_numpy(w).double() for w in wl.weights[4 * d:4 * d + 4]]
        a = torch.from_numpy(wl.x[0]).double() @ w_ih.T + torch.from_numpy(wl.h0[d]).double() @ w_hh.T + (b_ih + b_hh)
        i, f, g, _ = a.chunk(4, 1)
        want.append(torch.sigmoid(f) * torch.from_numpy(wl.c0[d]).double() + torch.sigmoid(i) * torch.tanh(g))
    want = torch.stack(want).numpy()
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    harness.forward(model, io)
    _, _, cT, _ = harness.results(io)
    rel = float(np.linalg.norm(cT - want) / np.linalg.norm(want))
    print("\n  case %r: cT %.3e" % (shape, rel), flush=True)
    assert rel <= bound
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    model.close()


@pytest.mark.parametrize("shape", [(0, 2, 2, 512, 512, 48, 72, 1), (1, 1, 1, 64, 256, 64, 300, 1)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d" % s[:7])
def test_reserved_steps_cover_fewer(gpu, shape):
    """Passes at the reserved number of steps, a launch of larger tiles at one: after rnn_model_reserve neither call allocates, so
    both can be recorded into a graph (which refuses to grow the workspace)."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg
    plans = [rnn.rnn_plan_query(c.cell, c.L, c.I, c.H, c.D, c.dtype, rnn.RNN_PLAN_AUTO, T, c.B, 256, 160 * 1024)[1] for T in (c.T, 1)]
    assert (plans[0]["col_tiles"], plans[0]["chains"]) == (1, 1) and plans[0]["col_blocks"] * 16 < c.B <= 16 * plans[1]["col_blocks"] * plans[1]["col_tiles"]
    print("\n  case %r" % (shape,), flush=True)
    warm, model, io = harness.DeviceModel(wl), harness.DeviceModel(wl), harness.DeviceIO(wl)
    for T in (1, c.T):                           # one-time set-up of the kernels
        assert rnn.rnn_forward(warm.handle, io.x, None, None, None, io.y, None, None, T, c.B, torch.cuda.current_stream()) == rnn.RNN_OK
    torch.cuda.synchronize()
    warm.close()
    assert rnn.rnn_model_reserve(model.handle, c.T, c.B) == rnn.RNN_OK
    held = rnn.rnn_model_device_bytes(model.handle)
    side = torch.cuda.Stream()
    for T in (1, c.T):
        def call(h, cc):
            return rnn.rnn_forward(model.handle, io.x, None, io.h0, io.c0, io.y, h, cc, T, c.B, torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            assert call(io.hT, io.cT) == rnn.RNN_OK
        want, wantc = torch.full_like(io.hT, 7.0), torch.full_like(io.cT, 7.0)
        assert call(want, wantc) == rnn.RNN_OK
        torch.cuda.synchronize()
        y = io.y[:T].clone()
        for _ in range(2):
            io.y.fill_(7.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(io.y[:T], y) and torch.equal(io.hT, want) and (c.cell == 1 or torch.equal(io.cT, wantc))
        del graph
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    assert rnn.rnn_model_device_bytes(model.handle) == held
    model.close()


@pytest.mark.parametrize("shape", [(0, 2, 1, 1024, 1024, 24, 2, 1), (1, 4, 1, 768, 768, 30, 1, 1), (0, 1, 1, 640, 640, 14, 1, 1), (0, 2, 1, 1024, 1024, 12, 258, 1),
                                   (0, 2, 1, 1024, 1024, 30, 300, 1), (0, 2, 1, 768, 768, 24, 64, 1), (0, 1, 2, 640, 640, 26, 40, 1)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d" % s[:7])
def test_reserved_steps_of_wide_layers_cover_fewer(gpu, shape):
    """Few sequences, or a last pass of few, through wide layers run on tagged words below a number of steps, and more of them on large
    tiles: rnn_model_reserve
    covers every smaller number of steps, and the results are those of a model that reserved nothing."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg
    kept, io, other = harness.DeviceModel(wl), harness.DeviceIO(wl), harness.DeviceIO(wl)
    assert rnn.rnn_model_reserve(kept.handle, c.T, c.B) == rnn.RNN_OK
    held = rnn.rnn_model_device_bytes(kept.handle)
    for T in sorted({1, 7, 8, 11, 12, 23, 24, c.T}):
        if T > c.T:
            continue
        print("\n  case %r: %d steps" % (shape, T), flush=True)
        fresh = harness.DeviceModel(wl)
        for m, o in ((kept, io), (fresh, other)):
            assert rnn.rnn_forward(m.handle, o.x, None, o.h0, o.c0, o.y, o.hT, o.cT, T, c.B, torch.cuda.current_stream()) == rnn.RNN_OK
        torch.cuda.synchronize()
        assert torch.equal(io.y[:T], other.y[:T]) and torch.equal(io.hT, other.hT)
        assert rnn.rnn_model_device_bytes(kept.handle) == held
        assert rnn.rnn_model_check(kept.handle) == rnn.RNN_OK
        fresh.close()
    kept.close()


def _call(rnn, model, io, T, B):
    import torch
    return rnn.rnn_forward(model.handle, io.x, None, io.h0, io.c0, io.y, io.hT, io.cT, T, B, torch.cuda.current_stream())


def _fewer_steps_find_their_workspace(gpu, shape, reset_before, reserved, steps):
    """Calls of `steps` after one of more steps, recorded into a graph (which refuses to grow the workspace): the bits of a model of
    their own, nothing allocated, and a graph of the longer call, recorded before them, still gives what it gave."""
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, False)
    c = wl.cfg

    def model_of():
        m = harness.DeviceModel(wl)
        assert rnn.rnn_model_set_gru_reset_before(m.handle, reset_before) == rnn.RNN_OK
        return m

    def recorded(m, io, T):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            rc = _call(rnn, m, io, T, c.B)
        assert rc == rnn.RNN_OK, "%d steps: %s" % (T, rnn.rnn_status_string(rc))
        return graph

    side = torch.cuda.Stream()
    kept, io, io_long, other = model_of(), harness.DeviceIO(wl), harness.DeviceIO(wl), harness.DeviceIO(wl)
    want = {}
    for T in steps:                              # (and the one-time set-up of the kernels)
        fresh = model_of()
        assert _call(rnn, fresh, other, T, c.B) == rnn.RNN_OK
        torch.cuda.synchronize()
        want[T] = (other.y[:T].clone(), other.hT.clone())
        fresh.close()
    if reserved:
        assert rnn.rnn_model_reserve(kept.handle, c.T, c.B) == rnn.RNN_OK
    assert _call(rnn, kept, io_long, c.T, c.B) == rnn.RNN_OK
    torch.cuda.synchronize()
    y, hT = io_long.y.clone(), io_long.hT.clone()
    held = rnn.rnn_model_device_bytes(kept.handle)
    long_graph = recorded(kept, io_long, c.T)
    for T in steps:
        print("\n  case %r: %d steps" % (shape, T), flush=True)
        graph = recorded(kept, io, T)
        for _ in range(2):
            io.y.fill_(7.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(io.y[:T], want[T][0]) and torch.equal(io.hT, want[T][1])
        assert _call(rnn, kept, io, T, c.B) == rnn.RNN_OK
        torch.cuda.synchronize()
        assert torch.equal(io.y[:T], want[T][0]) and torch.equal(io.hT, want[T][1])
        assert rnn.rnn_model_device_bytes(kept.handle) == held
        io_long.y.fill_(7.0)
        long_graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(io_long.y, y) and torch.equal(io_long.hT, hT)
        del graph
    assert rnn.rnn_model_check(kept.handle) == rnn.RNN_OK
    del long_graph
    kept.close()


@pytest.mark.parametrize("reserved", [True, False], ids=["reserved", "after_a_call"])
@pytest.mark.parametrize("shape,reset_before", [((1, 2, 1, 256, 256, 64, 9, 1), 0), ((1, 2, 1, 256, 256, 301, 16, 1), 1), ((0, 2, 1, 128, 128, 301, 3, 1), 0),
                                                ((0, 2, 2, 128, 128, 64, 18, 0), 0), ((0, 1, 1, 512, 512, 80, 20, 0), 0), ((0, 2, 1, 512, 512, 64, 5, 1), 0),
                                                ((1, 1, 1, 64, 256, 80, 300, 1), 0)],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_%s" % (s[:7] + ("f32" if s[7] == 0 else "bf16",)) if isinstance(s, tuple) else "rb%d" % s)
def test_slots_in_turn_cover_fewer_steps(gpu, shape, reset_before, reserved):
    """A state sequence uses few slots in turn from 16 steps on, and a slot for every step below: no fewer steps hold more."""
    _fewer_steps_find_their_workspace(gpu, shape, reset_before, reserved, (1, 15, 16, 17, 40, 63))


@pytest.mark.parametrize("reserved", [True, False], ids=["reserved", "after_a_call"])
@pytest.mark.parametrize("shape,steps", [((0, 2, 1, 1024, 1024, 8, 64, 1), (1, 5, 6, 7)), ((0, 4, 1, 1024, 1024, 30, 1, 1), (1, 7, 12, 23, 24)),
                                         ((0, 2, 2, 512, 512, 48, 72, 1), (1, 2, 4, 20)), ((0, 2, 1, 1024, 1024, 30, 300, 1), (1, 4, 8, 15)),
                                         ((0, 2, 1, 1024, 1024, 12, 258, 1), (1, 7, 8, 11)), ((0, 2, 2, 640, 640, 12, 3, 1), (1, 7, 8))],
                         ids=lambda s: "c%d_L%d_D%d_I%d_H%d_T%d_B%d_bf16" % s[:7] if len(s) == 8 else "to%d" % s[-1])
def test_another_plan_of_fewer_steps_finds_its_workspace(gpu, shape, steps, reserved):
    """Large tiles for a medium batch, tagged words for few sequences or a last pass of few."""
    _fewer_steps_find_their_workspace(gpu, shape, 0, reserved, steps)


@pytest.mark.parametrize("shape,digest", [((0, 2, 1, 1536, 1536, 24, 8, 1), "4ab4e57c91be3f6a"), ((1, 1, 1, 640, 1280, 20, 16, 1), "7776007b4d984933"),
                                          ((0, 1, 1, 1544, 1536, 12, 3, 1), "05ed68978cff64da"),
                                          ((0, 2, 1, 1024, 1024, 24, 4, 1), "f3f474cdc2c0e4ce"), ((1, 4, 1, 768, 768, 30, 1, 1), "38bee8ffcfaf741c"),
                                          ((0, 1, 1, 512, 1024, 12, 3, 1), "0f44c533d54e0b3d"), ((1, 2, 1, 1032, 640, 16, 4, 1), "3f3675137037fbc3"),
                                          ((0, 2, 2, 768, 768, 24, 4, 1), "d67e88dcb0a544aa")],
                         ids=["lstm_1536", "gru_1280_on_640", "lstm_1536_projected", "lstm_1024", "gru_768_one_sequence", "lstm_1024_on_512",
                              "gru_640_projected", "lstm_768_both_directions"])
def test_bits_of_the_tag_in_data_kernel(gpu, shape, digest):
    """Layers of 640 to 1536 units sum in the order of the tag-in-data kernel, which ran them first: its bits of y and hT."""
    import hashlib
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, True)
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    harness.forward(model, io)
    torch.cuda.synchronize()
    got = hashlib.sha256(io.y.view(torch.int16).cpu().numpy().tobytes() + io.hT.cpu().numpy().tobytes()).hexdigest()[:16]
    print("\n  case %r: %s" % (shape, got), flush=True)
    assert got == digest
    model.close()


def _with_options(rnn, wl, handle, clip):
    """Clipping, and for an LSTM peepholes from the workload's seed: what the model and an oracle are both given."""
    c = wl.cfg
    rng = np.random.default_rng(c.seed + 99)
    ps = [rng.uniform(-1, 1, (3, c.H)).astype(np.float32) for _ in range(c.L * c.D)] if c.cell == 0 else None
    assert rnn.rnn_model_set_clip(handle, clip) == rnn.RNN_OK
    if ps:
        assert rnn.rnn_model_set_peepholes(handle, ps, 0) == rnn.RNN_OK
    return ps


@pytest.mark.parametrize("shape,digest", [((0, 2, 1, 1024, 1024, 24, 3, 1), "0339149d51c5e864"), ((0, 4, 1, 768, 768, 30, 1, 1), "ad9396706a44a2cf"),
                                          ((0, 1, 1, 512, 1024, 12, 3, 1), "422428672fbb0355"), ((1, 2, 1, 640, 640, 16, 4, 1), "509f0e6722b16bb3")],
                         ids=["lstm_1024", "lstm_768_one_sequence", "lstm_1024_on_512", "gru_640"])
def test_bits_of_the_tag_in_data_kernel_with_options(gpu, oracle, shape, digest):
    """The same with peepholes (LSTM) and clipped gate arguments."""
    import hashlib
    import torch
    harness, rnn, W = gpu
    wl = _workload(W, shape, True)
    model, io = harness.DeviceModel(wl), harness.DeviceIO(wl)
    ps = _with_options(rnn, wl, model.handle, 0.3)
    harness.forward(model, io)
    torch.cuda.synchronize()
    assert rnn.rnn_model_check(model.handle) == rnn.RNN_OK
    _check(harness, wl, io, oracle.forward_workload(wl, nthreads=8, peepholes=ps, clip=0.3))
    got = hashlib.sha256(io.y.view(torch.int16).cpu().numpy().tobytes() + io.hT.cpu().numpy().tobytes()).hexdigest()[:16]
    print("\n  case %r: %s" % (shape, got), flush=True)
    assert got == digest
    model.close()
