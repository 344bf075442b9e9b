"""Host-side dispatch rules, without a GPU: which kernel a size goes to where both sides were measured."""
import ctypes

import pytest

from paper_1909_00562_amd import binding as bd


def _rule(symbol, restype, *argtypes):
    f = getattr(bd.load_library(), symbol)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


I32 = ctypes.c_int


@pytest.mark.parametrize("T, B, I, H, L, apart", [
    (50, 16, 512, 64, 1, True), (50, 16, 1024, 256, 1, True), (50, 16, 4096, 256, 1, True), (50, 16, 512, 1024, 1, True),
    (50, 128, 512, 512, 1, True), (50, 128, 1024, 1024, 1, True), (50, 128, 512, 256, 2, True),
    (50, 128, 1024, 512, 4, True), (50, 128, 4096, 1024, 2, True),
    (50, 16, 256, 128, 1, False), (50, 128, 512, 1024, 1, False), (10, 512, 512, 256, 1, False),
    (3, 128, 1024, 256, 1, False), (3, 128, 2048, 512, 2, False), (1, 128, 4096, 256, 1, False), (1, 128, 65536, 256, 1, False),
    (50, 128, 512, 512, 2, False),
    (50, 128, 512, 1024, 4, False), (50, 128, 1024, 1024, 4, False)])
def test_input_product_of_layer_0_where_it_was_faster(T, B, I, H, L, apart):
    """bf16: folded into the wavefronts or one product ahead of them, as measured at these sizes; fp32 always folded."""
    assert _rule("_ZN3asx14ls_input_apartItEEbiiiii", ctypes.c_bool, *[I32] * 5)(T, B, I, H, L) == apart
    assert not _rule("_ZN3asx14ls_input_apartIfEEbiiiii", ctypes.c_bool, *[I32] * 5)(T, B, I, H, L)
