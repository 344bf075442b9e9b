"""GPU parity of the stacked-LSTM entry points (lstm_stack_fwd / lstm_stack_bwd), called through the
C ABI, against the float64 oracle on the same seeded inputs.  Everything here needs an MI355X."""
import numpy as np
import pytest

import parity_util as pu
from oracle import lstm_stack_oracle as lo
from synth_inputs import make_lstm_inputs

pytestmark = pytest.mark.gpu


def _host(t):
    return t.detach().float().cpu().numpy()


def run_gpu(inp, use_states=True, **kw):
    import torch
    import paper_1909_00562_amd as lib
    d = lib.DeviceLstm(inp.x, inp.lengths, inp.W_ih, inp.W_hh, inp.b, inp.h0 if use_states else None,
                       inp.c0 if use_states else None, dtype=inp.dtype, dropout_p=getattr(inp, "dropout_p", 0.0),
                       dropout_seed=getattr(inp, "dropout_seed", 0), **kw)
    d.fwd()
    d.sync()
    f = dict(y=_host(d.y), hT=_host(d.hT), cT=_host(d.cT))
    dev = d.dev
    dy = torch.from_numpy(inp.dy).to(dev)
    dhT = torch.from_numpy(inp.dhT).to(dev) if use_states else None
    dcT = torch.from_numpy(inp.dcT).to(dev) if use_states else None
    d.bwd(dy, dhT, dcT)
    d.sync()
    g = dict(dx=_host(d.dx), dh0=_host(d.dh0), dc0=_host(d.dc0), dW_ih=[_host(t) for t in d.dW_ih],
             dW_hh=[_host(t) for t in d.dW_hh], db=[_host(t) for t in d.db])
    return f, g, d


def oracle_drop(inp):
    """Multipliers on the connections between the layers, [L-1, T, B, H] (None when dropout is off)."""
    p = getattr(inp, "dropout_p", 0.0)
    if p <= 0.0 or inp.L < 2:
        return None
    from oracle import train_extras_oracle as tx
    return tx.dropout_multiplier((inp.L - 1) * inp.T, inp.B, inp.H, p, inp.dropout_seed).reshape(
        inp.L - 1, inp.T, inp.B, inp.H)


def run_oracle(inp, use_states=True):
    fo = lo.forward(inp.x, inp.lengths, inp.W_ih, inp.W_hh, inp.b, inp.h0 if use_states else None,
                    inp.c0 if use_states else None, drop=oracle_drop(inp))
    go = lo.backward(fo, inp.dy, inp.dhT if use_states else None, inp.dcT if use_states else None)
    return fo, go


def compare(inp, f, g, fo, go, log=None):
    dt = inp.dtype
    valid = fo["valid"]
    assert np.all(f["y"][~valid] == 0.0), "output at padded steps"
    for k in ("y", "hT", "cT"):
        pu.assert_close(f[k], fo[k], dt, k, log)
    assert np.all(g["dx"][~valid] == 0.0), "dx at padded steps"
    for k in ("dx", "dh0", "dc0"):
        pu.assert_close(g[k], go[k], dt, k, log)
    for l in range(inp.L):
        for k in ("dW_ih", "dW_hh", "db"):
            pu.assert_close(g[k][l], go[k][l], dt, f"{k}[{l}]", log)


SHAPES = [
    # T, B, I, H, L
    (1, 1, 8, 8, 1),
    (6, 4, 24, 16, 3),
    (9, 5, 72, 40, 2),          # ragged against every tile edge
    (20, 32, 64, 128, 4),
    (7, 130, 40, 264, 2),       # more sentences than one 128-row tile
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_lstm_parity(shape, dtype):
    T, B, I, H, L = shape
    inp = make_lstm_inputs(T, B, I, H, L, seed=500 + T + B + H, dtype=dtype)
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_lstm_zero_length_sentences_and_default_states(dtype):
    inp = make_lstm_inputs(8, 6, 16, 24, 2, seed=77, dtype=dtype)
    inp.lengths[:] = [8, 0, 3, 12, -2, 1]                 # clamped to [0, T]
    f, g, _ = run_gpu(inp, use_states=False)
    fo, go = run_oracle(inp, use_states=False)
    compare(inp, f, g, fo, go)
    assert np.all(f["hT"][:, 1] == 0) and np.all(f["cT"][:, 4] == 0)      # never stepped: the zero initial state
    inp2 = make_lstm_inputs(8, 6, 16, 24, 2, seed=77, dtype=dtype)
    inp2.lengths[:] = [8, 0, 3, 12, -2, 1]
    f2, g2, _ = run_gpu(inp2)
    assert np.array_equal(f2["hT"][:, 1], inp2.h0[:, 1]) and np.array_equal(g2["dh0"][:, 4], inp2.dhT[:, 4])


def test_lstm_two_runs_are_bit_identical():
    inp = make_lstm_inputs(12, 16, 64, 64, 3, seed=5, dtype="bf16")
    f1, g1, _ = run_gpu(inp)
    f2, g2, _ = run_gpu(inp)
    for k in f1:
        assert np.array_equal(f1[k], f2[k]), k
    for k in ("dx", "dh0", "dc0"):
        assert np.array_equal(g1[k], g2[k]), k
    for l in range(inp.L):
        for k in ("dW_ih", "dW_hh", "db"):
            assert np.array_equal(g1[k][l], g2[k][l]), (k, l)


def _one_cell(a_o, c0):
    """y of one fp32 step whose forget gate is 1, input gate 0 and cell input -1: sigmoid(a_o) tanh(c0), [B, H]."""
    import torch
    import paper_1909_00562_amd as lib
    B, H = a_o.shape
    W_ih, b = np.zeros((4 * H, H), np.float32), np.zeros(4 * H, np.float32)
    W_ih[3 * H:] = np.eye(H, dtype=np.float32)          # the output gate's argument is x
    b[:H], b[H:2 * H], b[2 * H:3 * H] = -200, 200, -200
    d = lib.DeviceLstm(a_o[None], np.ones(B, np.int32), [W_ih], [np.zeros((4 * H, H), np.float32)], [b],
                       np.zeros((1, B, H), np.float32), c0[None], dtype="f32")
    d.fwd()
    d.sync()
    return _host(d.y)[0]


@pytest.mark.parametrize("lo, hi", [(1e-3, 0.1), (0.1, 0.6), (0.6, 0.7), (0.7, 1.5), (1.5, 9.0), (9.0, 18.0), (18.0, 86.0),
                                    (87.5, 103.0)])
def test_cell_functions_are_accurate_to_the_last_place(lo, hi):
    """Over every float the cell's sigmoid is off by 1.72 units of the last place at most and its tanh by 1.03 (1 / (1 + expf)
    and tanhf: 2.6 and 1.41), down to the subnormal results of sigmoid."""
    B, H = 256, 512
    rng = np.random.default_rng(int(hi * 10))
    a = rng.uniform(lo, hi, (B, H)).astype(np.float32)
    a[::2] *= -1
    ulp = lambda y, r: np.abs(y.astype(np.float64) - r) / np.spacing(np.abs(r).astype(np.float32)).astype(np.float64)
    big = np.full((B, H), 100.0, np.float32)
    sig = ulp(_one_cell(a, big), 1 / (1 + np.exp(-a.astype(np.float64))))
    tanh = ulp(_one_cell(2 * big, a), np.tanh(a.astype(np.float64)))
    assert sig.max() <= 1.72 and tanh.max() <= 1.04, (sig.max(), tanh.max())


def test_cell_functions_at_special_arguments():
    a = np.array([[0.0, -0.0, np.inf, -np.inf, np.nan, 1e38, -1e38, 1e-40, -1e-40, 104.5, -104.5, 88.0]], np.float32)
    big = np.full_like(a, 100.0)
    # (an infinite or NaN x meets the zeros of the other gates' weight rows, so sigmoid's come as finite ones)
    f = np.where(np.isfinite(a), a, 0)
    with np.errstate(over="ignore"):
        assert np.array_equal(_one_cell(f, big), (1 / (1 + np.exp(-f.astype(np.float64)))).astype(np.float32))
    y = _one_cell(2 * big, a)
    assert np.array_equal(y, np.tanh(a), equal_nan=True)
    number = ~np.isnan(a)
    assert np.array_equal(np.signbit(y[number]), np.signbit(a[number]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 7, 24, 40, 3),         # T, B, I, H, L: reductions of one and two steps
                                   (3, 97, 72, 1032, 2),      # 16 units x 32 sentences at one step
                                   (2, 225, 24, 648, 1),      # the same, more blocks than compute units
                                   (2, 385, 72, 1032, 1),     # 32 x 64
                                   (2, 97, 1000, 1024, 2),    # 16 x 32, six steps of the weight rows in flight
                                   (3, 21, 264, 328, 2),      # 16 x 16, six in layer 0, four in layer 1
                                   (4, 16, 256, 512, 2)])     # 16 x 16
def test_lstm_one_step_at_a_time_gives_the_bits_of_the_sequence(shape, dtype):
    """A decoder that advances the stack word by word from the states it got back follows the training pass exactly: one
    step reads the caller's weight rows, several read tiles of them, and both add in the same order."""
    T, B, I, H, L = shape
    inp = make_lstm_inputs(T, B, I, H, L, seed=H + B, dtype=dtype)
    inp.lengths[:] = T
    f, _, _ = run_gpu(inp)
    one = make_lstm_inputs(T, B, I, H, L, seed=H + B, dtype=dtype)
    one.T, one.lengths = 1, np.ones_like(inp.lengths)
    for t in range(T):
        one.x, one.dy = inp.x[t:t + 1].copy(), inp.dy[t:t + 1].copy()
        g, _, _ = run_gpu(one)
        assert np.array_equal(g["y"][0], f["y"][t]), t
        one.h0, one.c0 = g["hT"], g["cT"]
    assert np.array_equal(one.h0, f["hT"]) and np.array_equal(one.c0, f["cT"])


def test_lstm_paper_size_sixteen_sentences():
    """Table 2's model (embedding 512, hidden 1024, depth 4) at 50 steps, a batch of 16 sentences:
    everything, including the weight gradients, against the oracle."""
    inp = make_lstm_inputs(50, 16, 512, 1024, 4, seed=1909, dtype="bf16", min_len=20)
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    log = {}
    compare(inp, f, g, fo, go, log)
    print({k: (round(v["ratio"], 3), float(f"{v['norm']:.2e}")) for k, v in log.items()})


def test_lstm_paper_size_full_batch():
    """The configuration bench.py times (B = 128 at Table 2's size): every output and every gradient of the
    whole batch, weight gradients included, against the oracle run on the whole batch; the weight gradients of
    the batch must also equal the sum over 4 shards (fp32 summation order only)."""
    T, B, I, H, L = 50, 128, 512, 1024, 4
    inp = make_lstm_inputs(T, B, I, H, L, seed=50, dtype="bf16", min_len=20)
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)
    del fo, go
    acc = {k: [np.zeros_like(a, dtype=np.float64) for a in g[k]] for k in ("dW_ih", "dW_hh", "db")}
    q = B // 4
    for i in range(4):
        sl = slice(i * q, (i + 1) * q)
        sh = make_lstm_inputs(T, B, I, H, L, seed=50, dtype="bf16", min_len=20)
        sh.B = q
        sh.x, sh.lengths, sh.dy = inp.x[:, sl].copy(), inp.lengths[sl].copy(), inp.dy[:, sl].copy()
        sh.h0, sh.c0, sh.dhT, sh.dcT = (a[:, sl].copy() for a in (inp.h0, inp.c0, inp.dhT, inp.dcT))
        fs, gs, _ = run_gpu(sh)
        assert np.array_equal(fs["y"], f["y"][:, sl])           # a sentence does not see the batch around it
        for k in acc:
            for l in range(L):
                acc[k][l] += gs[k][l]
    for k in acc:
        for l in range(L):
            s = pu.err_stats(acc[k][l], g[k][l], "bf16")
            assert s["norm"] <= 5e-4, (k, l, s)


def test_encoder_decoder_attention_chain_fp32():
    """The interfaces fit: encoder LSTM -> decoder LSTM (initial state = the encoder's final state) ->
    attention-softmax forward/backward -> decoder backward -> encoder backward (which also receives the
    gradient of the decoder's initial state), fp32 storage, against the two oracles chained the same way."""
    import torch
    import paper_1909_00562_amd as lib
    from oracle import attn_softmax_oracle as orc
    from synth_inputs import make_custom
    S, T, B, I, H, L, V = 7, 6, 4, 12, 16, 2, 53
    enc_in = make_lstm_inputs(S, B, I, H, L, seed=31, dtype="f32")
    dec_in = make_lstm_inputs(T, B, I, H, L, seed=32, dtype="f32")
    att = make_custom(T=T, S=S, B=B, H=H, V=V, seed=33, dtype="f32", min_len=1)
    att.src_len = enc_in.lengths.copy()
    for b in range(B):                       # targets are padding exactly where the decoder's sentence has ended
        att.targets[:, b] = np.where(np.arange(T) < dec_in.lengths[b], np.maximum(att.targets[:, b], 1), att.pad_id)

    # oracle chain
    eo = lo.forward(enc_in.x, enc_in.lengths, enc_in.W_ih, enc_in.W_hh, enc_in.b)
    do = lo.forward(dec_in.x, dec_in.lengths, dec_in.W_ih, dec_in.W_hh, dec_in.b, eo["hT"], eo["cT"])
    args = (do["y"], eo["y"], att.src_len, att.W_a, att.W_c, att.W_out, att.b_out, att.targets, att.pad_id)
    fo = orc.forward(*args)
    go = orc.backward(*args, grad_scale=1.0)
    dgo = lo.backward(do, go["d_h_dec"])
    ego = lo.backward(eo, go["d_h_enc"], dgo["dh0"], dgo["dc0"])

    # GPU chain: device tensors handed from one entry point to the next
    enc = lib.DeviceLstm(enc_in.x, enc_in.lengths, enc_in.W_ih, enc_in.W_hh, enc_in.b, dtype="f32")
    dec = lib.DeviceLstm(dec_in.x, dec_in.lengths, dec_in.W_ih, dec_in.W_hh, dec_in.b, dtype="f32")
    enc.fwd()
    dec.h0, dec.c0 = enc.hT, enc.cT
    dec.fwd()
    db = lib.DeviceBatch(att)
    db.h_dec, db.h_enc = dec.y, enc.y
    db.fwd()
    db.bwd()
    dec.bwd(db.d_h_dec)
    enc.bwd(db.d_h_enc, dec.dh0, dec.dc0)
    enc.sync()
    assert int(db.n_tok.item()) == fo["n_tok"]
    assert abs(float(db.loss_sum.item()) - fo["loss_sum"]) <= 1e-4 * abs(fo["loss_sum"])
    pu.assert_close(_host(dec.dx), dgo["dx"], "f32", "decoder dx")
    pu.assert_close(_host(enc.dx), ego["dx"], "f32", "encoder dx")
    for l in range(L):
        pu.assert_close(_host(dec.dW_hh[l]), dgo["dW_hh"][l], "f32", f"decoder dW_hh[{l}]")
        pu.assert_close(_host(enc.dW_ih[l]), ego["dW_ih"][l], "f32", f"encoder dW_ih[{l}]")
        pu.assert_close(_host(enc.db[l]), ego["db"][l], "f32", f"encoder db[{l}]")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(6, 4, 24, 16, 3), (9, 5, 72, 40, 2), (20, 32, 64, 128, 4)])
def test_lstm_dropout_between_layers(shape, dtype):
    """Same words of the generator on both sides (the decision is integer work): with them every tensor
    agrees to the usual tolerance, and the run differs from the one without dropout."""
    T, B, I, H, L = shape
    inp = make_lstm_inputs(T, B, I, H, L, seed=900 + T + H, dtype=dtype)
    inp.dropout_p, inp.dropout_seed = 0.3, 20190900562 + T
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)
    plain = make_lstm_inputs(T, B, I, H, L, seed=900 + T + H, dtype=dtype)
    fp, _, _ = run_gpu(plain)
    assert not np.array_equal(fp["y"], f["y"])
    # rate 0 with a seed set is the same as no dropout, bit for bit
    zero = make_lstm_inputs(T, B, I, H, L, seed=900 + T + H, dtype=dtype)
    zero.dropout_p, zero.dropout_seed = 0.0, 77
    fz, gz, _ = run_gpu(zero)
    assert np.array_equal(fz["y"], fp["y"])


@pytest.mark.parametrize("shape", [(5, 7, 10, 219, 3), (4, 33, 9, 50, 2), (2, 3, 5, 3, 2)])
def test_lstm_dropout_of_widths_that_are_no_whole_vectors(shape):
    """fp32 rows of odd length: the masks of both passes are drawn an element at a time."""
    T, B, I, H, L = shape
    inp = make_lstm_inputs(T, B, I, H, L, seed=900 + T + H, dtype="f32")
    inp.dropout_p, inp.dropout_seed = 0.3, 20190900562 + T
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)


def test_lstm_dropout_paper_size_sixteen_sentences():
    inp = make_lstm_inputs(50, 16, 512, 1024, 4, seed=1910, dtype="bf16", min_len=20)
    inp.dropout_p, inp.dropout_seed = 0.3, 5
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)


@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_input_weight_saturates_its_gate(dtype, T):
    """The input x is exact in the storage type: an infinite weight of layer 0 makes a pre-activation +-inf, which the
    cell maps to a saturated gate, and never 0 * inf.  Every output stays finite and equal to the oracle's."""
    inp = make_lstm_inputs(T, 5, 24, 40, 2, seed=91, dtype=dtype)
    assert np.all(inp.x != 0)
    for gate, unit, k, sign in ((0, 3, 2, 1), (1, 17, 9, -1), (2, 39, 23, 1), (3, 0, 0, -1)):
        inp.W_ih[0][gate * 40 + unit, k] = sign * np.inf
    f, _, _ = run_gpu(inp)
    with np.errstate(over="ignore"):
        fo = lo.forward(inp.x, inp.lengths, inp.W_ih, inp.W_hh, inp.b, inp.h0, inp.c0)
    for key in ("y", "hT", "cT"):
        assert np.isfinite(fo[key]).all()
        pu.assert_close(f[key], fo[key], dtype, key)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("over", ["hT on h0", "y on x", "cT on c0", "hT past c0"])
def test_one_step_with_outputs_on_top_of_inputs(dtype, over):
    """A step in place gives the bits it gives into buffers of its own, whatever the order its blocks run in."""
    import torch
    import paper_1909_00562_amd as lib
    B, H, L = 37, 72, 3
    tdt, code = (torch.bfloat16, lib.AS_BF16) if dtype == "bf16" else (torch.float32, lib.AS_F32)
    g = torch.Generator(device="cuda").manual_seed(5)
    new = lambda *s: torch.randn(*s, generator=g, device="cuda")
    W_ih, W_hh = [[(new(4 * H, H) * 0.1).to(tdt) for _ in range(L)] for _ in range(2)]
    b = [new(4 * H).to(tdt) for _ in range(L)]
    x, h0, c0 = new(1, B, H).to(tdt), new(L, B, H), new(L, B, H)
    lengths = torch.randint(0, 2, (B,), generator=g, device="cuda", dtype=torch.int32)
    s = lib.LsShape(1, B, H, H, L, code, 0.0, 0)
    n = lib.lstm_stack_workspace_bytes(s)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")

    def run(x, h0, c0, y, hT, cT):
        lib.lstm_stack_fwd(s, x, lengths, W_ih, W_hh, b, h0, c0, y, hT, cT, ws, n)
        torch.cuda.synchronize()
        return [v.clone() for v in (y, hT, cT)]

    want = run(x, h0, c0, torch.empty_like(x), torch.empty_like(h0), torch.empty_like(c0))
    y, hT, cT = torch.empty_like(x), torch.empty_like(h0), torch.empty_like(c0)
    if over == "hT on h0":
        hT = h0
    elif over == "y on x":
        y = x
    elif over == "cT on c0":
        cT = c0
    else:
        both = torch.empty(L + 1, B, H, device="cuda")
        both[:L] = c0
        c0, hT = both[:L], both[1:]
    for got, w in zip(run(x, h0, c0, y, hT, cT), want):
        assert torch.equal(got, w)


@pytest.mark.parametrize("dtype, T, B, I, H, L", [("bf16", 9, 300, 520, 520, 2), ("f32", 3, 257, 72, 256, 2), ("f32", 9, 64, 67, 222, 2),
                                                  ("bf16", 3, 37, 24, 72, 3)])     # the last two: rows per position
@pytest.mark.parametrize("over", ["cT on c0", "cT past c0", "cT before c0", "cT past h0"])
def test_sequences_with_final_cells_on_top_of_initial_states(dtype, T, B, I, H, L, over):
    """cT anywhere over h0 and c0 gives the bits it gives in a buffer of its own; sentences without words among the others."""
    import torch
    import paper_1909_00562_amd as lib
    tdt, code = (torch.bfloat16, lib.AS_BF16) if dtype == "bf16" else (torch.float32, lib.AS_F32)
    g = torch.Generator(device="cuda").manual_seed(6)
    new = lambda *s: torch.randn(*s, generator=g, device="cuda")
    W_ih = [(new(4 * H, I if l == 0 else H) * 0.1).to(tdt) for l in range(L)]
    W_hh, b = [(new(4 * H, H) * 0.1).to(tdt) for _ in range(L)], [new(4 * H).to(tdt) for _ in range(L)]
    x, states = new(T, B, I).to(tdt), new(2, L, B, H)
    lengths = torch.randint(0, T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lengths[::5] = 0
    s = lib.LsShape(T, B, I, H, L, code, 0.0, 0)
    n = lib.lstm_stack_workspace_bytes(s)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    y, hT = torch.empty(T, B, H, dtype=tdt, device="cuda"), torch.empty(L, B, H, device="cuda")

    def run(h0, c0, cT):
        lib.lstm_stack_fwd(s, x, lengths, W_ih, W_hh, b, h0, c0, y, hT, cT, ws, n)
        torch.cuda.synchronize()
        return [v.clone() for v in (y, hT, cT)]

    want = run(states[0], states[1], torch.empty(L, B, H, device="cuda"))
    block = torch.empty(L + 1, B, H, device="cuda")
    first = over in ("cT before c0", "cT on c0")
    block[1 if first else 0:][:L] = states[0] if over == "cT past h0" else states[1]
    given, cT = block[1 if first else 0:][:L], block[1 if over == "cT on c0" or not first else 0:][:L]
    got = run(given, states[1], cT) if over == "cT past h0" else run(states[0], given, cT)
    for v, w in zip(got, want):
        assert torch.equal(v, w)


@pytest.mark.parametrize("dtype, T, B, I, H, L, dropout", [
    ("bf16", 9, 300, 520, 520, 2, 0.3),        # rows of words: more sentences than the block that numbers them has threads
    ("bf16", 33, 70, 264, 776, 2, 0.0),        # the gradient of x in a split product
    ("bf16", 60, 97, 1024, 208, 4, 0.0),       # in one that is not, and the input product ahead of the wavefronts
    ("bf16", 60, 97, 1024, 200, 3, 0.0),       # too little per word: rows per position
    ("bf16", 9, 37, 64, 1024, 4, 0.3),         # weight gradients of a kind of all layers in one launch
    # no whole vectors.  (With 219 units three of the 876 elements of db[1], sums over 37 sentences that no product here makes and
    # whose norm is right to 1.1e-7, lie so near zero that 1e-4 of them is less than their terms' rounding; 0.003 of them may.)
    ("f32", 21, 37, 67, 222, 2, 0.3),
    ("f32", 3, 257, 72, 256, 2, 0.0)])
@pytest.mark.parametrize("ends", ["mixed", "some empty", "all empty"])
def test_sequences_without_rows_for_padding(dtype, T, B, I, H, L, dropout, ends):
    """Weight gradients and the gradient of x over the words alone; sentences without a word keep their initial state."""
    inp = make_lstm_inputs(T, B, I, H, L, seed=H, dtype=dtype)
    inp.dropout_p, inp.dropout_seed = dropout, 5
    if ends == "some empty":
        inp.lengths[::3] = 0
        inp.lengths[1::7] = T
    elif ends == "all empty":
        inp.lengths[:] = 0
    f, g, _ = run_gpu(inp)
    fo, go = run_oracle(inp)
    compare(inp, f, g, fo, go)
    assert np.all(f["y"][np.arange(T)[:, None] >= inp.lengths[None, :]] == 0.0)
