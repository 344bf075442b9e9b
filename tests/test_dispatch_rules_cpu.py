"""Host-side dispatch rules, without a GPU: which kernel a size goes to where both sides were measured."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_1909_00562_amd import binding as bd


def _rule(symbol, restype, *argtypes):
    f = getattr(bd.load_library(), symbol)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


I32 = ctypes.c_int


@pytest.mark.parametrize("T, I, H, L, apart", [
    (50, 512, 64, 1, True), (50, 1024, 256, 1, True), (50, 4096, 256, 1, True), (50, 512, 512, 1, True),
    (50, 1024, 1024, 1, True), (10, 2048, 512, 1, True), (50, 512, 256, 2, True), (20, 2048, 512, 2, True),
    (50, 1024, 512, 4, True),
    (50, 256, 128, 1, False), (50, 512, 1024, 1, False), (10, 512, 256, 1, False), (3, 1024, 256, 1, False),
    (3, 2048, 512, 2, False), (1, 4096, 256, 1, False), (1, 65536, 256, 1, False), (50, 512, 512, 2, False),
    (50, 512, 1024, 4, False), (50, 1024, 1024, 2, False)])
def test_input_product_of_layer_0_where_it_was_faster(T, I, H, L, apart):
    """bf16: folded into the wavefronts or one product ahead of them, as measured at these sizes; fp32 always folded.  The
    number of sentences is no argument: a sentence's result does not depend on its batch."""
    assert _rule("_ZN3asx14ls_input_apartItEEbiiii", ctypes.c_bool, *[I32] * 4)(T, I, H, L) == apart
    assert not _rule("_ZN3asx14ls_input_apartIfEEbiiii", ctypes.c_bool, *[I32] * 4)(T, I, H, L)


@pytest.mark.parametrize("dtype, T, B, I, H, L, packed", [
    ("t", 50, 64, 512, 1024, 4, True), ("t", 64, 192, 256, 256, 4, True), ("t", 40, 64, 512, 640, 2, True), ("t", 32, 128, 512, 512, 1, True),
    ("t", 64, 192, 64, 128, 2, False), ("t", 60, 128, 256, 256, 2, False), ("t", 32, 64, 512, 512, 1, False),
    ("t", 64, 12, 64, 1024, 1, False), ("t", 1, 16384, 512, 1024, 4, False), ("t", 50, 16385, 512, 1024, 4, False),
    ("f", 30, 64, 256, 512, 2, True), ("f", 24, 48, 256, 384, 2, True), ("f", 10, 64, 256, 384, 1, True),
    ("f", 60, 128, 64, 128, 2, False), ("f", 30, 64, 192, 192, 1, False), ("f", 24, 16, 256, 384, 1, False)])
def test_rows_of_words_where_they_were_faster(dtype, T, B, I, H, L, packed):
    assert _rule(f"_ZN3asx9ls_packedI{dtype}EEbiiiii", ctypes.c_bool, *[I32] * 5)(T, B, I, H, L) == packed


@pytest.mark.parametrize("S, H, fused", [(1, 1, True), (64, 4096, True), (65, 256, True), (128, 256, True), (65, 257, False), (128, 2048, False),
                                         (129, 64, False)])
def test_f32_attention_in_one_launch_where_it_was_faster(S, H, fused):
    assert _rule("_ZN3asx24attn_f32_fused_supportedEii", ctypes.c_bool, I32, I32)(S, H) == fused


def _plan(M, N, K, batch, bf16, allow_split=True, multi_segment=False, counted=False):
    """(tile, splits) of a product: tile 0 = 128 x 128, 1 = 256 x 256, 2 = 64 x 64 (bf16)."""
    f = _rule("_ZN3asx9gemm_planEiiiibbbb", ctypes.c_uint64, *[I32] * 4, *[ctypes.c_bool] * 4)
    v = f(M, N, K, batch, bf16, allow_split, multi_segment, counted)
    return v & 0xffffffff, v >> 32


def _plan_of(which, N, H, bf16=True):
    """The same for h_c ("hc") or the last product of d_h_dec ("dh") of N rows; tile 3 = the kernel for few rows."""
    v = _rule(f"_ZN3asx7plan_{which}Eiib", ctypes.c_uint64, I32, I32, ctypes.c_bool)(N, H, bf16)
    return v & 0xffffffff, v >> 32


FEW_ROWS_HC = [(1, 456), (16, 472), (17, 504), (113, 512), (127, 456)]     # (rows, units), the edges of its rows among them


@pytest.mark.parametrize("N, H", FEW_ROWS_HC)
def test_h_c_of_few_rows_goes_to_the_kernel_for_few_rows(N, H):
    assert _plan_of("hc", N, H) == (3, 1)
    assert _plan_of("hc", N, H, bf16=False)[0] != 3


@pytest.mark.parametrize("N, H", [(1, 448), (114, 512), (128, 456), (1, 520), (40, 576), (16, 1024)])
def test_h_c_of_other_sizes_stays_with_the_tiles(N, H):
    assert _plan_of("hc", N, H)[0] != 3


@pytest.mark.parametrize("N, H, few", [
    (1, 64, True), (128, 256, True), (32, 512, True), (17, 640, True), (128, 768, True), (1, 1024, True), (128, 1024, True),
    (33, 512, False), (128, 512, False), (40, 640, False), (33, 264, False), (129, 1024, False), (1, 1032, False)])
def test_d_h_dec_of_few_rows_where_the_kernel_for_few_rows_was_faster(N, H, few):
    assert (_plan_of("dh", N, H)[0] == 3) == few
    assert _plan_of("dh", N, H, bf16=False)[0] != 3


def _f32_split_bound(M, N, K, batch):
    tiles = -(-M // 64) * -(-N // 64) * batch
    if tiles >= 384:
        return 1
    slices = -(-K // 16)
    most = min(-(-768 // tiles), slices // 16, 32)
    return 1 if most <= 1 else -(-slices // -(-slices // most))


def test_f32_products_keep_their_sums_in_fp64():
    """A split's partial sum is rounded to fp32, so no product gets more splits than the bound; none is left without
    reduction tiles."""
    rng = random.Random(7)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    sizes = [(512, 512, 496, 1), (32, 64, 1000, 1), (16, 2048, 32000, 1), (30, 20000, 4096, 1), (1, 1, 1, 1)]
    sizes += [(log(1, 8192), log(1, 8192), log(1, 65536), rng.choice((1, 1, 2))) for _ in range(20000)]
    for s in sizes:
        _, splits = _plan(*s, bf16=False)
        assert 1 <= splits <= _f32_split_bound(*s), s
        tiles = -(-s[2] // 32)
        assert -(-tiles // splits) * (splits - 1) < tiles, s
    assert _plan(512, 512, 496, 1, bf16=False)[1] == 1


@pytest.mark.parametrize("M, N, K, batch, plan", [
    (2048, 2048, 16384, 1, (1, 4)), (2048, 2048, 16384, 2, (1, 2)), (2048, 2048, 7680, 2, (1, 2)),
    (1024, 1024, 12800, 2, (1, 8)), (4096, 1024, 12800, 1, (1, 4)), (6144, 512, 6400, 1, (1, 5)),
    (1280, 1024, 32000, 1, (1, 12)), (3776, 512, 27403, 1, (1, 8)),
    (4096, 1024, 6400, 1, (0, 1)), (8192, 512, 6400, 1, (0, 1)), (2048, 2048, 4096, 1, (0, 1)), (1024, 1024, 6400, 1, (2, 1)), (4096, 1024, 3200, 1, (0, 1)),
    (1536, 1536, 2560, 1, (0, 1)), (16000, 512, 1286, 1, (0, 1)), (4096, 4096, 4096, 1, (1, 1))])
def test_bf16_tile_that_was_the_faster_one(M, N, K, batch, plan):
    """Weight-gradient products (and dlogits W_out) whose time was taken with every tile and split: 256 x 256 tiles above,
    the smaller ones below."""
    assert _plan(M, N, K, batch, bf16=True) == plan


@pytest.mark.parametrize("M, N, K, plan", [(800, 1024, 32000, (0, 9)), (8192, 512, 8000, (0, 1)), (8000, 512, 8192, (0, 2)),
                                           (128000, 2048, 16384, (1, 1)), (6400, 1024, 32000, (1, 5))])
def test_bf16_tile_where_the_device_counts_the_size(M, N, K, plan):
    """Row compaction: the sizes are bounds, about half of which is there; smaller tiles win earlier."""
    assert _plan(M, N, K, 1, bf16=True, counted=True) == plan


@pytest.mark.parametrize("N, V, H, leaves", [
    (16, 16000, 512, True), (179, 2054, 128, True), (128, 32000, 1024, True), (1024, 2003, 64, True), (1025, 2003, 64, False),
    (182, 51130, 128, False),
    (16, 2097144, 1280, True), (16, 2097145, 1280, False),     # rows of 2^21 and more: past the vector write-out
    (16, 2200000, 640, False), (1, 4000000, 512, False), (64, 4000000, 1024, False)])
def test_softmax_statistics_from_the_projection_where_its_kernels_make_them(N, V, H, leaves):
    assert _rule("_ZN3asx23projection_leaves_statsEiii", ctypes.c_bool, *[I32] * 3)(N, V, H) == leaves


@pytest.mark.parametrize("V, H, past", [(32000, 1024, True), (32000, 512, True), (131073, 64, True), (131072, 64, False),
                                        (16000, 512, False), (1000, 64, False)])
def test_gradients_past_the_caches_where_dw_out_is_larger_than_they_are(V, H, past):
    assert _rule("_ZN3asx21gradients_past_cachesEii", ctypes.c_bool, I32, I32)(V, H) == past


@pytest.mark.parametrize("V, H, past", [(6000, 1280, True), (4000, 1536, True), (1, 2048, True), (2, 2047, False), (1200, 1728, False), (2292, 1024, False)])
def test_gradients_past_the_caches_where_all_of_them_are_larger_still(V, H, past):
    assert _rule("_ZN3asx21gradients_past_cachesEii", ctypes.c_bool, I32, I32)(V, H) == past


@pytest.mark.parametrize("edge, form, M, N, laced", [
    (128, "TN", 1024, 1024, True), (128, "NN", 2257, 1000, True), (64, "NT", 128, 1024, True), (64, "TN", 1024, 1024, True),
    (128, "NT", 6400, 1024, True), (128, "NT", 600, 8000, True), (128, "NN", 6400, 1024, True), (64, "NT", 6400, 1024, True),
    (64, "NN", 8192, 1024, True),
    (128, "TN", 16000, 512, False), (128, "TN", 9000, 640, False), (128, "TN", 4096, 2048, False), (64, "TN", 2048, 768, False),
    (64, "TN", 4096, 1024, False)])
def test_fragment_reads_between_matrix_instructions_where_they_were_faster(edge, form, M, N, laced):
    """64 x 64 and 128 x 128 tiles, measured with the reads of a reduction tile ahead of its matrix instructions and between
    those of the tile before: no size may be slower than with the reads ahead."""
    f = _rule("_ZN3asx15gemm_tile_lacedEbl", ctypes.c_bool, ctypes.c_bool, ctypes.c_int64)
    assert f(form[0] == "N", -(-M // edge) * -(-N // edge)) == laced


@pytest.mark.parametrize("T, S, B, H, V, dtype, skip", [
    (5, 53, 103, 32, 27126, bd.AS_F32, 1), (11, 27, 45, 31, 28054, bd.AS_F32, 0), (10, 123, 55, 22, 25179, bd.AS_F32, 0),
    (2, 39, 241, 2281, 197, bd.AS_F32, 1), (78, 29, 53, 92, 2017, bd.AS_F32, 0)])
def test_static_scratch_holds_shapes_just_below_its_size(T, S, B, H, V, dtype, skip):
    """attn_softmax_fwd_static takes a shape by the size of its whole workspace, so that must not grow with parts of the
    backward pass that are never alive together."""
    shape = bd.AsShape(T, S, B, H, V, 0, dtype, 1.0, 0.0, 0, skip)
    assert bd.attn_softmax_workspace_bytes(shape) <= bd.AS_STATIC_SCRATCH_BYTES


def test_workspace_of_the_largest_training_step():
    """64 steps x 256 sentences, 2048 units, 128000 words: the column sums of dlogits (262 MB) and the partial sums share
    their place."""
    shape = bd.AsShape(64, 64, 256, 2048, 128000, 0, bd.AS_BF16, 1.0, 0.0, 0, 1)
    assert bd.attn_softmax_workspace_bytes(shape) <= 6.45e9


def test_workspace_of_one_lstm_step():
    """A decoder's call (T = 1, 128 sentences, four layers of 1024 units) reads the caller's weights; the backward pass of
    such a step needs tiles of four weights at a time, not of seven."""
    shape = bd.LsShape(1, 128, 512, 1024, 4, bd.AS_BF16, 0.0, 0)
    assert bd.load_library().lstm_stack_workspace_bytes(ctypes.byref(shape)) <= 64 << 20


@pytest.mark.parametrize("K, H, six", [
    (256, 256, True), (256, 320, True), (320, 320, True), (256, 384, True), (1024, 1024, True), (1088, 1088, True),
    (64, 64, False), (128, 128, False), (384, 384, False), (256, 448, False), (448, 448, False), (256, 512, False),
    (640, 640, False), (704, 704, False), (768, 768, False), (896, 896, False), (256, 1024, False), (1280, 1280, False)])
def test_lstm_one_step_has_six_steps_of_weight_rows_in_flight_where_that_was_faster(K, H, six):
    """Four or six steps ahead, both measured at these widths: no layer-step may be slower than with four."""
    assert _rule("_ZN3asx22ls_row_steps_in_flightEii", ctypes.c_int, I32, I32)(K, H) == (6 if six else 4)


def test_lstm_workspace_has_no_partial_sums_for_products_that_are_not_split():
    """12800 rows, four layers of 1024 units: alone each weight gradient would be split in four (67 MB of partial sums); in
    one launch for all layers none is, and those of dx (64 wide, 13 MB) are the largest left."""
    T, B, I, H, L = 100, 128, 64, 1024, 4
    assert _plan(4 * H, H, T * B, 1, bf16=True)[1] == 4
    shape = bd.LsShape(T, B, I, H, L, bd.AS_BF16, 0.0, 0)
    dx = 4 * T * B * I * 4
    gates_and_states = L * T * B * 4 * H * 4 + L * (T + 1) * B * H * (4 + 2) + (L - 1) * T * B * H * 2
    backward = L * T * B * 4 * H * 2 + dx + 2 * L * 4 * H * B * 2 + (2 * L - 1) * 4 * H * H * 2   # dG, its tiles, the weights'
    assert bd.load_library().lstm_stack_workspace_bytes(ctypes.byref(shape)) <= gates_and_states + backward + (8 << 20)


HIP_STUB = """
#pragma once
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 1 };
enum { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
extern int device, calls, fail;
inline hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { ++calls; return fail ? hipErrorUnknown : hipSuccess; }
"""
LDS_LIMIT_MAIN = """
#include "lds_limit.h"
int device = 0, calls = 0, fail = 0;
int main() {
  asx::LdsLimit a, b;
  auto expect = [](bool ok) { if (!ok) __builtin_trap(); };
  expect(a.raise(0, 1) == hipSuccess && calls == 1);
  expect(a.raise(0, 1) == hipSuccess && calls == 1);     // once per device
  device = 1;
  expect(a.raise(0, 1) == hipSuccess && calls == 2);     // another device of the same process
  expect(b.raise(0, 1) == hipSuccess && calls == 3);     // another kernel
  device = 2; fail = 1;
  expect(a.raise(0, 1) == hipErrorUnknown && calls == 4);
  fail = 0;
  expect(a.raise(0, 1) == hipSuccess && calls == 5);     // a failure is not remembered
  device = 70;
  expect(a.raise(0, 1) == hipSuccess && a.raise(0, 1) == hipSuccess && calls == 7);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_lds_limit_is_raised_on_every_device(tmp_path):
    """The limit of a kernel's dynamic LDS belongs to the device it is loaded on: host code against a stub of the runtime."""
    csrc = os.path.join(os.path.dirname(bd.library_path()), "csrc")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_STUB)
    (tmp_path / "main.cpp").write_text(LDS_LIMIT_MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-std=c++17", f"-I{tmp_path}", f"-I{csrc}", str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True)
    # and every launcher that needs more than 64 KiB goes through it
    for name in os.listdir(csrc):
        if name != "lds_limit.h":
            assert "hipFuncSetAttribute" not in open(os.path.join(csrc, name)).read(), name
