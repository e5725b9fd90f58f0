"""The forward passes that users of this library run, as a list to measure: listed(), and draw() for more of the same.

A case is one model shape and one call shape:
    cell         "lstm" | "gru"
    dtype        "bf16" | "f32"       storage type of x, y and the weights
    L, D, I, H   layers, directions, input width, hidden width
    T, B         steps and sequences of the call
    len_min      0: every sequence has T steps; else lengths are uniform in [len_min, T], x is zero behind them
    h0           whether an initial state is handed in
    layout       "time" [T, B, .] | "batch" [B, T, .]
    extra        "" | "peephole_clip" (LSTM) | "reset_before" (GRU, the ONNX default form)
"""
import math

import torch

from paper_2307_11339_amd import rnn


def _case(name, cell, dtype, L, D, I, H, T, B, len_min=0, h0=False, layout="time", extra=""):
    c = dict(cell=cell, dtype=dtype, L=L, D=D, I=I, H=H, T=T, B=B, len_min=len_min, h0=h0, layout=layout, extra=extra)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One new frame of a live stream through a kept model: the state of the call before comes in, the new one goes
        # out.  The smallest call there is; all of it is latency.
        _case("stream_step", "lstm", "bf16", 4, 1, 1024, 1024, 1, 1, h0=True),
        # The named workload C1: a small sensor model on one short sequence, plain fp32.
        _case("small_f32", "lstm", "f32", 1, 1, 64, 128, 32, 1),
        # C2: an online batch of a few requests through a GRU.
        _case("online_gru", "gru", "bf16", 2, 1, 256, 512, 100, 8, h0=True),
        # C3: one sequence through a deep LSTM, as in interactive speech or text.
        _case("one_sequence", "lstm", "bf16", 4, 1, 1024, 1024, 128, 1),
        # C4: a bidirectional encoder on padded sequences of very different lengths.
        _case("bidirectional", "lstm", "bf16", 2, 2, 512, 512, 256, 64, len_min=64),
        # C5: offline encoding of a full batch, the throughput case and the largest call.
        _case("offline_encoder", "lstm", "bf16", 8, 1, 1024, 1024, 512, 256),
        # The middle of the paper's model grid: many narrow layers in fp32.
        _case("deep_narrow_f32", "lstm", "f32", 12, 1, 64, 64, 96, 8),
        # A batch of an fp32 model, as it comes out of training without conversion.
        _case("batch_f32", "lstm", "f32", 2, 1, 512, 512, 128, 64),
        # An acoustic encoder: 80 features a frame, a width and sizes that fit nothing, padded batch-first tensors.
        _case("acoustic_ragged", "lstm", "bf16", 3, 2, 80, 320, 301, 57, len_min=75, layout="batch"),
        # A batch that is not a power of two and larger than one launch takes at this width.
        _case("odd_batch", "lstm", "bf16", 2, 1, 1024, 1024, 64, 300),
        # A wide model on a few requests.
        _case("wide_few", "lstm", "bf16", 2, 1, 1536, 1536, 128, 8),
        # A GRU as ONNX files hold it by default: the reset gate acts before the candidate's recurrent product.
        _case("onnx_gru", "gru", "bf16", 2, 1, 256, 256, 64, 16, extra="reset_before"),
    ]


def _log(rng, lo, hi, step=1):
    """A size in [lo, hi], even over its logarithm, a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999)))
    return min(hi - hi % step, max(lo + -lo % step, int(v / step + 0.5) * step))


def _one(rng):
    """One draw: a kind of use as in listed(), its sizes spread over that use's range."""
    use = rng.choice(("stream", "latency", "grid_f32", "batch_f32", "bidirectional", "throughput", "wide", "onnx_gru"))
    cell, dtype, D, len_min, h0, layout, extra = "lstm" if rng.random() < 0.7 else "gru", "bf16", 1, 0, False, "time", ""
    if use == "stream":
        dtype = rng.choice(("bf16", "bf16", "f32"))
        L, H, T, B, h0 = rng.randint(1, 6), _log(rng, 64, 1024 if dtype == "bf16" else 512, 8), _log(rng, 1, 8), _log(rng, 1, 16), True
    elif use == "latency":
        L, H, T, B, h0 = rng.randint(1, 6), _log(rng, 128, 1024, 8), _log(rng, 16, 256), _log(rng, 1, 16), rng.random() < 0.3
    elif use == "grid_f32":
        cell, dtype, L, H, T, B = "lstm", "f32", rng.randint(2, 16), _log(rng, 32, 128, 4), _log(rng, 32, 128), _log(rng, 1, 16)
    elif use == "batch_f32":
        dtype, D = "f32", rng.choice((1, 1, 2))
        L, H, T, B = rng.randint(1, 3), _log(rng, 64, 640, 4), _log(rng, 32, 160), _log(rng, 16, 128)
    elif use == "bidirectional":
        D, L, H, T, B = 2, rng.randint(1, 4), _log(rng, 128, 768, 8), _log(rng, 64, 400), _log(rng, 8, 128)
        layout = rng.choice(("time", "batch"))
    elif use == "throughput":
        L, H, T, B = rng.randint(1, 6), _log(rng, 256, 1024, 8), _log(rng, 64, 400), _log(rng, 32, 512)
    elif use == "wide":
        L, H, T, B = rng.randint(1, 3), _log(rng, 1032, 2048, 8), _log(rng, 32, 160), _log(rng, 1, 64)
    else:
        cell, dtype, extra = "gru", rng.choice(("bf16", "bf16", "f32")), "reset_before"
        L, H, T, B = rng.randint(1, 3), _log(rng, 64, 512, 8), _log(rng, 16, 96), _log(rng, 1, 64)
    # the input of most stacks is as wide as the layers; the rest have a feature vector of their own
    I = H if rng.random() < 0.5 else _log(rng, 40, 1024, 8)
    if use in ("batch_f32", "bidirectional", "throughput") and rng.random() < 0.6:
        len_min = max(1, T // 4)
    if not extra and cell == "lstm" and rng.random() < 0.1:
        extra = "peephole_clip"
    return _case("", cell, dtype, L, D, I, H, T, B, len_min, h0, layout, extra)


def draw(rng):
    while True:
        c = _one(rng)
        # no more arithmetic than a fraction of the largest listed pass: such widths run at a fraction of its rate
        most = 4e12 if c["dtype"] == "bf16" else 8e9 if c["extra"] == "reset_before" else 1.2e11
        if work(dict(c, len_min=0))["flops"] <= most:
            return c


def _sizes(c):
    return 4 if c["cell"] == "lstm" else 3, [c["I"]] + [c["D"] * c["H"]] * (c["L"] - 1), 2 if c["dtype"] == "bf16" else 4


class _State:
    """The model and the device tensors of one user."""

    def __init__(self):
        self.model = None

    def __del__(self):
        if self.model is not None:
            torch.cuda.synchronize()
            rnn.rnn_model_destroy(self.model)


def prepare(case, seed):
    c, s = case, _State()
    gates, widths, _ = _sizes(c)
    L, D, H, T, B = c["L"], c["D"], c["H"], c["T"], c["B"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(k, *shape):
        return torch.empty(shape, device="cuda").uniform_(-k, k, generator=g)

    k, weights = H ** -0.5, []
    for l in range(L):
        for _ in range(D):
            weights += [uniform(k, gates * H, widths[l]).to(dt), uniform(k, gates * H, H).to(dt),
                        uniform(k, gates * H).to(dt), uniform(k, gates * H).to(dt)]
    torch.cuda.synchronize()
    s.model = rnn.rnn_model_create(rnn.RNN_LSTM if c["cell"] == "lstm" else rnn.RNN_GRU, L, c["I"], H, D,
                                   rnn.RNN_BF16 if c["dtype"] == "bf16" else rnn.RNN_F32, weights, 1)
    said = [rnn.rnn_model_set_batch_first(s.model, int(c["layout"] == "batch"))]
    if c["extra"] == "peephole_clip":
        peepholes = [uniform(1.0, 3, H) for _ in range(L * D)]
        torch.cuda.synchronize()
        said += [rnn.rnn_model_set_peepholes(s.model, peepholes, 1), rnn.rnn_model_set_clip(s.model, 3.0)]
    elif c["extra"] == "reset_before":
        said.append(rnn.rnn_model_set_gru_reset_before(s.model, 1))
    said.append(rnn.rnn_model_reserve(s.model, T, B))
    if any(rc != rnn.RNN_OK for rc in said):
        raise RuntimeError("the model could not be set up: %r" % (said,))

    def layout(t):  # from time-major
        return t.transpose(0, 1).contiguous() if c["layout"] == "batch" else t

    x = torch.randn((T, B, c["I"]), generator=g, device="cuda")
    s.lengths = None
    if c["len_min"]:
        s.lengths = torch.randint(c["len_min"], T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
        x *= (torch.arange(T, device="cuda")[:, None] < s.lengths[None, :])[:, :, None]
    s.x = layout(x.to(dt))
    lstm = c["cell"] == "lstm"
    state = (L * D, B, H)
    s.h0 = torch.randn(state, generator=g, device="cuda") * 0.1 if c["h0"] else None
    s.c0 = torch.randn(state, generator=g, device="cuda") * 0.1 if c["h0"] and lstm else None
    s.y = layout(torch.empty((T, B, D * H), dtype=dt, device="cuda"))
    s.hT = torch.empty(state, device="cuda")
    s.cT = torch.empty(state, device="cuda") if lstm else None
    s.T, s.B = T, B
    return s


def run(s):
    rc = rnn.rnn_forward(s.model, s.x, s.lengths, s.h0, s.c0, s.y, s.hT, s.cT, s.T, s.B, torch.cuda.current_stream())
    if rc != rnn.RNN_OK:
        raise rnn.RnnError(rc, "rnn_forward")
    return [s.y, s.hT] if s.cT is None else [s.y, s.hT, s.cT]


def work(case):
    """Every weight, input and state read once, every output written once; the two products of every cell that a
    sequence really has (half the padding of uniform lengths is nobody's work)."""
    c = case
    gates, widths, size = _sizes(c)
    L, D, H, T, B = c["L"], c["D"], c["H"], c["T"], c["B"]
    cells = B * ((T + c["len_min"]) / 2 if c["len_min"] else T)
    products = sum(gates * H * D * (w + H) for w in widths)
    lstm = 2 if c["cell"] == "lstm" else 1
    return {"bytes": products * size + 2 * L * D * gates * H * size  # weights and biases
            + cells * c["I"] * size + T * B * D * H * size          # x, y
            + lstm * L * D * B * H * 4 * (2 if c["h0"] else 1),     # states
            "flops": 2.0 * cells * products}


def tolerance(case):
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
