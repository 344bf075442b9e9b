"""GPU parity at the sizes where a dispatch rule changes its mind or a tile has a remainder, against the float64
oracle.  Everything here needs an MI355X."""
import numpy as np
import pytest

import parity_util as pu
from synth_inputs import make_custom

pytestmark = pytest.mark.gpu


def _parity(inp, skip=False):
    run = pu.GpuRun(inp, skip_pad_rows=skip)
    f, g = run.fwd(), run.bwd()
    fo, go = pu.run_oracle(inp)
    pu.compare_all(f, g, fo, go, inp.dtype, pad_rows_hold=inp.pad_id if skip else None)


@pytest.mark.parametrize("shape", [(1, 9, 5, 584, 301), (5, 6, 8, 712, 203)])
def test_h_c_split_with_ragged_segments(shape):
    """h_c = tanh(W_c [ctx; h_dec]) is split along a reduction of three segments, each of ceil(H / 64) tiles: hidden
    sizes for which 3 * ceil(H / 64) and ceil(3 * H / 64) differ enough to leave a split without tiles."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=H, dtype="bf16", min_len=1, pad_prob=0.1))


@pytest.mark.parametrize("shape", [(1, 3, 1, 136, 2003), (2, 4, 8, 264, 2003), (1, 5, 17, 328, 2003), (4, 6, 32, 512, 2003),
                                   (3, 6, 43, 504, 2003)])
def test_h_c_of_few_rows(shape):
    """1 to 129 rows that need no split: one 64 x 64 tile of rows to three, reductions that end inside a tile."""
    T, S, B, H, V = shape
    inp = make_custom(T=T, S=S, B=B, H=H, V=V, seed=H, dtype="bf16", min_len=1, pad_prob=0.1)
    inp.dropout_p, inp.dropout_seed = 0.3, 11
    _parity(inp)


@pytest.mark.parametrize("shape", [(1, 3, 1, 456, 2003),      # one row; a reduction that ends inside a line
                                   (2, 4, 8, 472, 2003),      # 16 rows, the last of one block form; columns past a block
                                   (1, 5, 17, 504, 2003),     # 17, the first of the other
                                   (1, 6, 113, 512, 2003),    # the most rows of the longest reduction
                                   (1, 4, 127, 456, 2003),    # the most rows
                                   (1, 4, 128, 456, 2003)])   # one more: tiles
def test_h_c_by_the_kernel_for_few_rows(shape):
    """The sizes of test_h_c_of_few_rows_goes_to_the_kernel_for_few_rows: three segments, tanh, dropout and the saved
    derivative."""
    T, S, B, H, V = shape
    inp = make_custom(T=T, S=S, B=B, H=H, V=V, seed=H + B, dtype="bf16", min_len=1, pad_prob=0.1)
    inp.dropout_p, inp.dropout_seed = 0.3, 11
    _parity(inp)


@pytest.mark.parametrize("shape", [(32, 512), (33, 264), (128, 256), (128, 776), (33, 1024)])   # rows, units
def test_d_h_dec_of_few_rows(shape):
    """dQ W_a^T added to d_h_dec by the kernel for few rows, and (33 x 264) by tiles."""
    B, H = shape
    _parity(make_custom(T=1, S=7, B=B, H=H, V=2003, seed=H + B, dtype="bf16", min_len=1))


@pytest.mark.parametrize("shape", [(1, 97, 72, 1032, 2)])      # T, B, I, H, L: 260 blocks, 66 of the largest form
def test_lstm_one_step_in_blocks_of_16_units_and_32_sentences(shape):
    """The form a decoder step of the largest model takes, with ragged edges in units, sentences and input."""
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    T, B, I, H, L = shape
    # (1024 and 768: 256 and 192 blocks, one per compute unit at most, with six and four steps of the weight rows in flight)
    for units in (H, H - 8, H - 8 * 33):
        inp = make_lstm_inputs(T, B, I, units, L, seed=units, dtype="bf16")
        f, g, _ = tl.run_gpu(inp)
        fo, go = tl.run_oracle(inp)
        tl.compare(inp, f, g, fo, go)


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("shape", [(20, 5, 13, 60, 16003),     # 64 x 64 tiles of logits and dW_out, ragged in every direction
                                   (3, 33, 11, 121, 999),      # rows that are not 16-byte aligned: scalar loads
                                   (31, 7, 3, 132, 2051)])     # split reductions with a remainder
def test_f32_products_at_tile_edges(shape, skip):
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V, dtype="f32", min_len=1, pad_prob=0.3), skip)


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("shape", [(1, 5, 65, 72, 321),        # one row and one column past a 64 x 64 tile, H of 9 vectors
                                   (2, 33, 64, 136, 1000),     # whole row tiles, reductions of 2 and a bit tiles
                                   # source barely over one tile.  (With a vocabulary as small as 67 the rounding of
                                   # dlogits to bf16 leaves 59 elements of dW_out to the row-scale floor, in the
                                   # 128 x 128 kernel just as many; the budget of 0.0022 was taken at larger ones.)
                                   (9, 70, 7, 200, 643)])
def test_bf16_products_in_64x64_tiles(shape, skip):
    """Few output tiles: the 64 x 64 kernel in its three operand forms, with remainders in rows, columns and reduction."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=H, dtype="bf16", min_len=1, pad_prob=0.2), skip)


@pytest.mark.parametrize("shape", [(1, 1, 3, 8, 67),          # one step, one source position, one reduction step
                                   # (The vocabulary of the larger ones: with 203 words the rounding of dlogits to bf16
                                   # leaves 0.019 to 0.028 of dW_out to the row-scale floor, whatever made the states;
                                   # the budget of 0.0022 was taken at larger ones.)
                                   (16, 32, 4, 72, 515),      # whole row and source tiles, a reduction of 2 steps and a bit
                                   (17, 33, 3, 520, 203),     # one past them; waves with one and two pairs of steps
                                   (33, 64, 5, 1032, 2003),   # waves with two and three pairs
                                   (19, 65, 3, 136, 203),     # 32-column slots
                                   (3, 128, 2, 2056, 203),    # the longest source, waves with four and five pairs
                                   (31, 20, 192, 24, 2003),    # 32 decoder steps per workgroup, a source of one tile
                                   (33, 45, 97, 40, 2003)])    # the same, of two
def test_fused_attention_at_tile_edges(shape):
    """bf16, S <= 128: 16 or 32 decoder steps and 32, 64 or 128 source positions per workgroup, eight waves that share the
    reduction and the columns; one sentence of length 0.  (Wide states get weights of 0.05, as in the largest configuration:
    with 0.1 the scores of 1032 units are twice those the tolerance was taken at, and the rounding of dQ alone moves an
    element of d_h_dec to 1.34 of it.)"""
    T, S, B, H, V = shape
    inp = make_custom(T=T, S=S, B=B, H=H, V=V, seed=S, dtype="bf16", min_len=1, pad_prob=0.1, w=0.05 if H > 1000 else 0.1)
    inp.src_len[B // 2] = 0
    _parity(inp)


@pytest.mark.parametrize("shape", [(33, 64, 5, 1032, 2003), (3, 128, 2, 2056, 2003)])
def test_fused_attention_of_wide_states_with_large_weights(shape):
    """The same widths with the weights of the narrower ones, scores twice as large."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=S, dtype="bf16", min_len=1, pad_prob=0.1, w=0.1))


@pytest.mark.parametrize("T, S, B", [(9, 5, 120), (33, 5, 97), (9, 40, 120), (33, 40, 97), (9, 100, 120)])   # 16 steps a workgroup, 32
def test_fused_attention_without_a_list_or_a_count_to_clear(T, S, B):
    """More than 1024 rows, padding rows not left out: the forward pass has nothing but the attention to do."""
    _parity(make_custom(T=T, S=S, B=B, H=72, V=8011, seed=S, dtype="bf16", min_len=1, pad_prob=0.1))


def test_fused_attention_of_more_steps_than_a_grid_has_blocks():
    """S > 64 takes 16 decoder steps per workgroup: 16 * 65536 + 64 steps need more workgroups than a grid may have in one
    direction.  Every step repeats the one 64 before it, so its results do too, bit for bit."""
    import torch
    import paper_1909_00562_amd as lib
    from paper_1909_00562_amd import binding as bd
    P = 64
    T = 16 * 65536 + P
    inp = make_custom(T=P, S=65, B=1, H=8, V=8, seed=1, dtype="bf16", min_len=1, pad_prob=0.1)
    results = lambda db: [db.view(bd.AS_VIEW_ALPHA)[0], db.view(bd.AS_VIEW_CTX)[:, 0], db.d_h_dec[:, 0]]
    few = lib.DeviceBatch(inp)
    few.fwd(), few.bwd(), few.sync()
    first = [v.float() for v in results(few)]
    inp.h_dec, inp.targets = np.tile(inp.h_dec, (T // P, 1, 1)), np.tile(inp.targets, (T // P, 1))
    inp.T = T
    db = lib.DeviceBatch(inp)
    db.fwd(), db.bwd(), db.sync()
    for v, f in zip(results(db), first):
        rows = v.reshape(T // P, P, -1)
        assert torch.equal(rows, rows[:1].expand_as(rows))
        assert torch.allclose(rows[0].float(), f, rtol=1e-2, atol=1e-3)


@pytest.mark.parametrize("dtype, H", [("bf16", 72), ("bf16", 520), ("f32", 68), ("f32", 67)])   # f32, 67: no whole vectors
@pytest.mark.parametrize("pad_prob", [0.0, 0.3, 0.97])         # all rows, some, a row or two of 35
def test_split_dz_goes_straight_to_its_rows(dtype, H, pad_prob):
    """Few rows, a long vocabulary: dlogits W_out is a split product, whose combine step also undoes the row compaction."""
    inp = make_custom(T=5, S=6, B=7, H=H, V=4099, seed=H, dtype=dtype, min_len=1, pad_prob=pad_prob)
    _parity(inp, skip=True)


def test_lstm_f32_largest_block_in_vectors():
    """16 units x 32 sentences in fp32 with a hidden size of whole vectors (other sizes: test_lstm_wavefronts_at_block_edges)."""
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    inp = make_lstm_inputs(4, 65, 24, 1028, 4, seed=1028, dtype="f32")
    f, g, _ = tl.run_gpu(inp)
    fo, go = tl.run_oracle(inp)
    tl.compare(inp, f, g, fo, go)


@pytest.mark.parametrize("shape", [(70, 5, 200, 643),          # a second sweep over the source positions
                                   (131, 3, 264, 997),         # more than the fused kernel takes forward
                                   (1500, 2, 512, 777)])       # many sweeps
def test_one_step_attention_backward(shape):
    """T = 1, bf16: one workgroup per sentence, 64 source positions at a time."""
    S, B, H, V = shape
    _parity(make_custom(T=1, S=S, B=B, H=H, V=V, seed=S, dtype="bf16", min_len=1))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 1, 8, 8, 2),            # one sentence
                                   (5, 33, 40, 200, 3),        # units and sentences past every block shape
                                   (4, 65, 24, 1032, 2),       # remainders in 16 units x 32 sentences forward
                                   # 32 units x 64 sentences forward, 64 x 32 backward (fp32: 16 x 32 both ways): the
                                   # largest blocks, from four (three) layers in one launch on, with remainders
                                   (5, 65, 24, 1032, 4),
                                   # one step: the caller's weight rows, widths of whole vectors.  (c = f c0 + i g is
                                   # rounded at 2^-24 of its terms, 6e-8: elements of y below 6e-4, about one in a
                                   # thousand, need the row-scale floor; a tensor of 1275 admits one, this one four.)
                                   (1, 65, 16, 72, 2),
                                   (1, 9, 24, 1032, 4)])        # one step, tiles of one wavefront's weights at a time
def test_lstm_wavefronts_at_block_edges(shape, dtype):
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    T, B, I, H, L = shape
    if dtype == "f32" and T > 1:
        I, H = I + 1, H + 3     # widths that are no multiple of four
    inp = make_lstm_inputs(T, B, I, H, L, seed=H, dtype=dtype)
    f, g, _ = tl.run_gpu(inp)
    fo, go = tl.run_oracle(inp)
    tl.compare(inp, f, g, fo, go)


@pytest.mark.parametrize("dtype, I, H", [("bf16", 72, 1032), ("f32", 36, 1028)])
def test_lstm_one_step_in_the_largest_blocks(dtype, I, H):
    """The caller's weight rows in 32 units x 64 sentences (fp32: 16 x 32), rows that end inside a line."""
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    inp = make_lstm_inputs(1, 385, I, H, 2, seed=H, dtype=dtype)
    f, g, _ = tl.run_gpu(inp)
    fo, go = tl.run_oracle(inp)
    tl.compare(inp, f, g, fo, go)


def test_lstm_weight_gradients_of_all_layers_at_once():
    """dW_hh of five layers in one launch (180 tiles of 256 x 256, ragged in rows and columns), dW_ih one by one."""
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    inp = make_lstm_inputs(2, 3, 16, 712, 5, seed=712, dtype="bf16")
    f, g, _ = tl.run_gpu(inp)
    fo, go = tl.run_oracle(inp)
    tl.compare(inp, f, g, fo, go)


@pytest.mark.parametrize("states", [True, False])
@pytest.mark.parametrize("shape", [(16, 21, 648, 72, 1),       # a wide x: its product ahead of the wavefronts, ragged tiles
                                   (8, 33, 1032, 40, 3),       # with layers above it
                                   (4, 65, 2064, 520, 2),      # in 16 units x 32 sentences
                                   (4, 65, 2064, 1032, 4)])    # in 32 units x 64 sentences
def test_lstm_wide_input(shape, states):
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    T, B, I, H, L = shape
    inp = make_lstm_inputs(T, B, I, H, L, seed=I, dtype="bf16")
    f, g, _ = tl.run_gpu(inp, use_states=states)
    fo, go = tl.run_oracle(inp, use_states=states)
    tl.compare(inp, f, g, fo, go)


@pytest.mark.parametrize("skip", [False, True])
def test_static_scratch_just_below_its_size(skip):
    """The forward pass in the library's own scratch, nearly all of it used, and the passes that share one area of a
    caller's workspace, against the oracle."""
    import test_zz_no_alloc as na
    inp = make_custom(T=5, S=53, B=103, H=32, V=27126, seed=5, dtype="f32", min_len=1, pad_prob=0.2)
    na._run_pair(inp, skip)
    _parity(inp, skip)


def test_lstm_wide_input_does_not_see_its_batch():
    """With the input product ahead of the wavefronts too, a sentence's outputs are the same bits in every batch: 130
    sentences and 16 go to different tiles of that product and different blocks."""
    import test_gpu_lstm as tl
    from synth_inputs import make_lstm_inputs
    inp = make_lstm_inputs(10, 130, 1032, 512, 2, seed=3, dtype="bf16")
    f, _, _ = tl.run_gpu(inp)
    part = make_lstm_inputs(10, 130, 1032, 512, 2, seed=3, dtype="bf16")
    for k in ("x", "dy"):
        setattr(part, k, np.ascontiguousarray(getattr(part, k)[:, 32:48]))
    for k in ("h0", "c0", "dhT", "dcT"):
        setattr(part, k, np.ascontiguousarray(getattr(part, k)[:, 32:48]))
    part.lengths, part.B = part.lengths[32:48].copy(), 16
    g, _, _ = tl.run_gpu(part)
    assert np.array_equal(g["y"], f["y"][:, 32:48])
    assert np.array_equal(g["hT"], f["hT"][:, 32:48]) and np.array_equal(g["cT"], f["cT"][:, 32:48])


@pytest.mark.parametrize("shape", [(1, 9, 3, 8, 643),          # one reduction tile, one row tile
                                   (1, 7, 65, 136, 643),       # a row past a tile, a reduction of two tiles and a bit
                                   (6, 20, 43, 520, 2003)])    # ragged in every direction
def test_both_gradients_through_w_c_in_one_launch(shape):
    """dC = dz W_c[:, :H] with dz as value and remainder (bf16 pair out), dz W_c[:, H:] of the value alone (float out)."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V + H, dtype="bf16", min_len=1, pad_prob=0.1))


@pytest.mark.parametrize("shape", [(6, 7, 55, 520, 3003),      # 64 x 64: logits, and dW_out with its fragments read first
                                   (9, 5, 45, 520, 8011),      # 128 x 128: the same
                                   # (With 643 words 0.011 of dW_out need the row-scale floor, in the other loop as
                                   # many, 3630 elements; the budget of 0.0022 was taken at larger vocabularies.)
                                   (10, 6, 103, 520, 3003)])   # both gradients through W_c in one launch, 306 blocks
def test_bf16_products_with_several_blocks_per_compute_unit(shape):
    """More than 256 blocks of 64 x 64 or 128 x 128 tiles, reductions of fewer tiles than the ring has stages among them (the
    attention products and dW_a of the last)."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V + H, dtype="bf16", min_len=1, pad_prob=0.1))


@pytest.mark.parametrize("shape", [(1, 9, 3, 72, 2003),        # two products behind dQ, fewer blocks than the XCDs share evenly
                                   (5, 6, 7, 136, 2003),       # three, 9 + 3 + 21 blocks of ragged tiles
                                   # more than 256 blocks; dW_c the one with the longer reduction.  (With 2003 words the
                                   # rounding of dlogits to bf16 leaves 0.0030 of dW_out, a product of its own, to the
                                   # row-scale floor; the budget of 0.0022 was taken at larger vocabularies.)
                                   (30, 7, 61, 264, 8011),
                                   (2, 7, 61, 520, 2003)])     # dC and dH1 the one
def test_bf16_products_of_a_pass_in_one_launch(shape):
    """dW_c with dC and dH1, and dW_a with d_h_dec and d_h_enc, blocks of one product behind those of another."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V + H, dtype="bf16", min_len=1, pad_prob=0.1))


@pytest.mark.parametrize("shape", [(1, 7, 20, 64, 131101), (3, 7, 100, 136, 70003), (9, 7, 100, 136, 70003)])
def test_bf16_gradients_past_the_caches(shape):
    """dW_out of more than 32 MiB in 64 x 64 tiles with dz, in 128 x 128 with dz in either; dW_c and dW_a of the same calls,
    in launches of up to 256 blocks and of more, d_h_enc beside the latter."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V + H, dtype="bf16", min_len=1, pad_prob=0.1))


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("shape", [(3, 8, 5, 36, 517),         # whole vectors in every product; tiles of a few rows
                                   (5, 7, 6, 68, 517),         # but in the source positions
                                   (5, 7, 6, 67, 517),         # none
                                   (9, 12, 31, 132, 1031)])    # splits, several blocks per compute unit
def test_f32_products_of_a_pass_in_one_launch(shape, skip):
    """dW_out with dz, dW_c with dC and dH1, dW_a with d_h_dec and d_h_enc, blocks of one product behind those of another."""
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V + H, dtype="f32", min_len=1, pad_prob=0.2), skip)


@pytest.mark.parametrize("dtype, S", [("bf16", 5), ("bf16", 129), ("f32", 5)])     # beside either form of the attention
@pytest.mark.parametrize("T, B", [(1, 1), (3, 171), (64, 64), (241, 17), (723, 17)])   # 4096 positions at a time: 4096, 4097, 12291
def test_list_of_word_positions(T, B, dtype, S):
    """Row compaction: words numbered in increasing position, -1 at padding (compared by fwd), and the outputs at padding."""
    inp = make_custom(T=T, S=S, B=B, H=8, V=11, seed=T, dtype=dtype, min_len=1, pad_prob=0.4)
    f = pu.GpuRun(inp, skip_pad_rows=True).fwd()
    pad = inp.targets == inp.pad_id
    assert np.array_equal(f["tgt_mask"].astype(bool), ~pad) and f["n_tok"] == int((~pad).sum())
    assert np.all(f["tok_loss"][pad] == 0.0) and np.all(f["argmax"][pad] == inp.pad_id)


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("N, H, V", [(1, 64, 67), (16, 64, 643), (17, 64, 643), (130, 72, 2003),     # 64 x 64 tiles
                                     (70, 520, 16003), (128, 1024, 20005)])                          # 128 x 128
def test_statistics_from_the_projection(N, H, V, skip):
    """lse, argmax and loss of few rows against those of the logits as stored, in double.  Words that the bias rules out (-inf):
    more than a tile of them, and the last.  Bound of lse: the sum of V terms, 32 and then 4, 64 and V / 4096 at a time, has a
    relative error below 105 * 2^-24, every exponential one of 2^-23 and its argument's rounding, below |x - m| log2(e) 2^-24 for
    terms of that weight: 1.2e-5, and 2e-6 for rounding lse itself; the loss the same again for its rounding."""
    import torch
    inp = make_custom(T=1, S=5, B=N, H=H, V=V, seed=V + N, dtype="bf16", min_len=1, pad_prob=0.2)
    inp.b_out = inp.b_out.copy()
    inp.b_out[1:min(V // 2, 150)] = -np.inf
    inp.b_out[V - 1] = -np.inf
    inp.targets[inp.targets != inp.pad_id] = V - 2
    import paper_1909_00562_amd as lib
    from paper_1909_00562_amd import binding as bd
    db = lib.DeviceBatch(inp, skip_pad_rows=skip)
    db.fwd(), db.sync()
    live = (db.targets.reshape(-1) != inp.pad_id)
    rows = int(live.sum()) if skip else N
    x = db.view(bd.AS_VIEW_LOGITS).reshape(N, -1)[:rows].double()
    assert bool(torch.isneginf(x[:, V - 1]).all())
    lse = torch.logsumexp(x, 1)
    assert torch.allclose(db.view(bd.AS_VIEW_LSE).reshape(-1)[:rows].double(), lse, rtol=0, atol=1.4e-5)
    best = torch.argmax((x == x.max(1, keepdim=True).values).int(), 1).int()      # the lowest that attains it
    arg, loss = db.argmax.reshape(-1), db.tok_loss.reshape(-1).double()
    want = lse - x[:, V - 2]
    if skip:
        assert torch.equal(arg[live], best) and torch.allclose(loss[live], want, rtol=0, atol=1.6e-5)
        want_sum = want.sum()
    else:
        assert torch.equal(arg, best) and torch.allclose(loss[live], want[live], rtol=0, atol=1.6e-5)
        want_sum = want[live].sum()
    assert bool((loss[~live] == 0).all()) and int(db.n_tok.item()) == int(live.sum())
    assert abs(float(db.loss_sum.item()) - float(want_sum)) <= 1.6e-5 * max(1, int(live.sum())) + 2 ** -23 * abs(float(want_sum))


@pytest.mark.parametrize("step", [False, True])
def test_more_words_than_whole_vectors_reach(step):
    """2200000 words, 640 units: a projection in 64 x 64 tiles that writes its logits element by element.  Logits against double
    products at some words, the last among them, as rounded to bf16; lse against that of the logits as stored.  Bound of lse: a
    thread adds at most V / 256 terms one after the other, 8594 * 2^-24 = 5.2e-4 relative, and then a few hundred sums and
    roundings of single terms, below 3e-5."""
    import torch
    import paper_1909_00562_amd as lib
    from paper_1909_00562_amd import binding as bd
    N, S, H, V, pad = 16, 5, 640, 2200000, 0
    g = torch.Generator(device="cuda").manual_seed(21)
    new = lambda *s: torch.rand(*s, generator=g, device="cuda").mul_(0.2).sub_(0.1).bfloat16()
    out = lambda *s, dtype=torch.float32: torch.zeros(*s, dtype=dtype, device="cuda")
    h, he, W_a, W_c, W_out, b_out = new(N, H), new(S, N, H), new(H, H), new(H, 2 * H), new(V, H), new(V)
    src_len = torch.full((N,), S, dtype=torch.int32, device="cuda")
    targets = torch.randint(1, V, (N,), generator=g, device="cuda", dtype=torch.int32)
    targets[0], targets[1] = V - 1, pad
    loss_sum, n_tok, tok_loss, argmax = out(1), out(1, dtype=torch.int32), out(N), out(N, dtype=torch.int32)
    attn_mask, tgt_mask = out(N, S, dtype=torch.uint8), out(N, dtype=torch.uint8)
    shape = lib.AsShape(1, S, N, H, V, pad, lib.AS_BF16, 1.0)
    n = (lib.attn_softmax_step_workspace_bytes if step else lib.attn_softmax_workspace_bytes)(shape)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    if step:
        lib.attn_softmax_step_prepare(shape, he, W_a, ws, n)
        lib.attn_softmax_step_fwd(shape, h, he, src_len, W_c, W_out, b_out, targets, loss_sum, n_tok, tok_loss, argmax, ws, n)
    else:
        lib.attn_softmax_fwd(shape, h, he, src_len, W_a, W_c, W_out, b_out, targets, loss_sum, n_tok, tok_loss, argmax,
                             attn_mask, tgt_mask, ws, n)
    torch.cuda.synchronize()

    def view(which):
        addr, nbytes, ld = lib.attn_softmax_view(shape, ws, which)
        return ws[addr - ws.data_ptr():addr - ws.data_ptr() + nbytes], ld

    raw, ld = view(bd.AS_VIEW_LOGITS)
    logits = raw.view(torch.bfloat16).view(N, ld)[:, :V]
    h_c = view(bd.AS_VIEW_HC)[0].view(torch.bfloat16).view(N, H)
    words = torch.cat([torch.arange(130, device="cuda"), torch.arange(V - 130, V, device="cuda"),
                       torch.randint(0, V, (4096,), generator=g, device="cuda")])
    want = h_c.double() @ W_out[words].double().T + b_out[words].double()
    assert torch.allclose(logits[:, words].double(), want, rtol=2 ** -8, atol=1e-5)
    x = logits.double()
    lse = torch.logsumexp(x, 1)
    assert torch.allclose(view(bd.AS_VIEW_LSE)[0].view(torch.float32).double(), lse, rtol=0, atol=6e-4)
    assert torch.equal(argmax.long(), torch.argmax((x == x.max(1, keepdim=True).values).int(), 1))
    live = targets != pad
    loss = (lse - x[torch.arange(N, device="cuda"), targets.long()])[live]
    assert torch.allclose(tok_loss[live].double(), loss, rtol=0, atol=6e-4) and float(tok_loss[1]) == 0.0
    assert int(n_tok.item()) == N - 1 and abs(float(loss_sum.item()) - float(loss.sum())) <= 6e-4 * N


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 3, 4, 67),          # one step, one source position, a quarter of a reduction step
                                   (16, 16, 4, 64, 131),      # whole tiles; a reduction step per wave
                                   (17, 17, 3, 260, 131),     # one past them; a remainder of columns
                                   (5, 33, 6, 67, 131),       # no whole vectors
                                   (35, 64, 2, 141, 131),
                                   (3, 65, 5, 36, 131),
                                   (18, 64, 2, 1028, 131),    # several sweeps over the columns
                                   (18, 128, 2, 256, 131),    # the longest source, one whole sweep
                                   (18, 128, 2, 1028, 131), (3, 65, 2, 257, 131),   # more of both: separate launches
                                   (4, 129, 3, 36, 131)])     # one more: separate launches
def test_f32_fused_attention_at_tile_edges(shape, skip):
    """fp32, S <= 64, or S <= 128 and H <= 256: 16 decoder steps and 16 to 128 source positions per workgroup; one sentence of length 0."""
    T, S, B, H, V = shape
    inp = make_custom(T=T, S=S, B=B, H=H, V=V, seed=S + H, dtype="f32", min_len=1, pad_prob=0.1, w=0.05 if H > 1000 else 0.1)
    inp.src_len[B // 2] = 0
    _parity(inp, skip)


@pytest.mark.parametrize("entry, S", [("fwd", 5), ("fwd", 129), ("step", 5)])     # the three kernels ahead of the statistics
@pytest.mark.parametrize("skip", [False, True])
def test_loss_sum_of_further_calls_on_a_workspace(entry, S, skip):
    """Rows in several blocks, of which the last adds up the losses: every call finds one.  The sum is of floats in double, rounded once."""
    import torch
    import paper_1909_00562_amd as lib
    N, H, V, pad = 130, 72, 2003, 0
    g = torch.Generator(device="cuda").manual_seed(3)
    new = lambda *s: torch.rand(*s, generator=g, device="cuda").mul_(0.2).sub_(0.1).bfloat16()
    h, he, W_a, W_c, W_out, b_out = new(N, H), new(S, N, H), new(H, H), new(H, 2 * H), new(V, H), new(V)
    src_len = torch.full((N,), S, dtype=torch.int32, device="cuda")
    loss_sum, n_tok = torch.empty(1, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    tok_loss, argmax = torch.empty(N, device="cuda"), torch.empty(N, dtype=torch.int32, device="cuda")
    shape = lib.AsShape(1, S, N, H, V, pad, lib.AS_BF16, 1.0, 0.0, 0, 1 if skip else 0)
    n = (lib.attn_softmax_step_workspace_bytes if entry == "step" else lib.attn_softmax_workspace_bytes)(shape)
    ws = torch.full((n,), 0x5a, dtype=torch.uint8, device="cuda")
    if entry == "step":
        lib.attn_softmax_step_prepare(shape, he, W_a, ws, n)
    for words in (N, 77, 0, 129):
        targets = torch.randint(1, V, (N,), generator=g, device="cuda", dtype=torch.int32)
        targets[words:] = pad
        loss_sum.fill_(float("nan")), n_tok.fill_(-1), tok_loss.fill_(float("nan"))
        if entry == "step":
            lib.attn_softmax_step_fwd(shape, h, he, src_len, W_c, W_out, b_out, targets, loss_sum, n_tok, tok_loss, argmax, ws, n)
        else:
            lib.attn_softmax_fwd(shape, h, he, src_len, W_a, W_c, W_out, b_out, targets, loss_sum, n_tok, tok_loss, argmax,
                                 None, None, ws, n)
        torch.cuda.synchronize()
        want = float(tok_loss.double().sum())
        assert int(n_tok.item()) == words and bool((tok_loss[words:] == 0).all())
        assert abs(float(loss_sum.item()) - want) <= 2 ** -23 * abs(want) and (want > words or words == 0)


@pytest.mark.parametrize("shape, alone", [((5, 6, 7, 136, 2003), False), ((64, 64, 256, 2048, 1003), True)])
def test_stage_times_of_products_with_and_without_a_launch_of_their_own(shape, alone):
    """A product in a launch of its own is timed under its own stage, products that share one under the first one's."""
    import paper_1909_00562_amd as lib
    T, S, B, H, V = shape
    db = lib.DeviceBatch(make_custom(T=T, S=S, B=B, H=H, V=V, seed=1, dtype="bf16", min_len=1, w=0.05))
    lib.attn_softmax_profile_enable(True)
    try:
        db.fwd(), db.bwd(), db.sync()
        launches = {k: v["launches"] for k, v in lib.attn_softmax_profile_read().items()}
    finally:
        lib.attn_softmax_profile_enable(False)
    got = {k: launches[k] for k in ("gemm_dwout", "gemm_dhc", "gemm_dwc", "gemm_dch", "gemm_dwa", "gemm_dh", "attn_bwd", "misc")}
    # attn_bwd: the first half in one kernel, and d_h_enc; misc: the sum of the losses, and the column sums of dlogits
    assert got == dict(gemm_dwout=1, gemm_dhc=int(alone), gemm_dwc=1, gemm_dch=2 * alone, gemm_dwa=1, gemm_dh=int(alone),
                       attn_bwd=1 + alone, misc=2 * alone)
