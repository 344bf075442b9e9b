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


@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("shape", [(20, 5, 13, 60, 16003),     # 64 x 64 tiles of logits and dW_out, ragged in every direction
                                   (3, 33, 11, 121, 999),      # rows that are not 16-byte aligned: scalar loads
                                   (31, 7, 3, 132, 2051)])     # split reductions with a remainder
def test_f32_products_at_tile_edges(shape, skip):
    T, S, B, H, V = shape
    _parity(make_custom(T=T, S=S, B=B, H=H, V=V, seed=V, dtype="f32", min_len=1, pad_prob=0.3), skip)
