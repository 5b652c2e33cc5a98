"""Host-side checks of the C ABI (no GPU): the library loads, exports every symbol that
include/ocs.h declares, and rejects bad arguments before any device work."""
import ctypes as C
import os
import re
import struct

import msgpack
import numpy as np
import pytest

from oracle import ref
from paper_1901_09504_amd import binding as B
from paper_1901_09504_amd.build import LIB

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "ocs.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ocs_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared()
    assert {"ocs_num_splits", "ocs_split_weights", "ocs_quantize", "ocs_split_act", "ocs_qgemm",
            "ocs_select_channels", "ocs_workspace_bytes", "ocs_strerror"} <= set(names)
    L = B.lib()
    for n in names:
        assert hasattr(L, n), n
        assert hasattr(B, n) or n in ("ocs_strerror", "ocs_last_hip_error"), f"binding lacks {n}"


def _kernels():
    """What the compiler noted about every kernel of the built library: the AMDGPU metadata notes of its code objects."""
    data, at, kernels = open(LIB, "rb").read(), 0, []
    while (at := data.find(b"AMDGPU\0\0", at)) >= 0:
        name, size, kind = struct.unpack_from("<III", data, at - 12)
        if (name, kind) == (7, 32):
            kernels += msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]
        at += 8
    return kernels


# Kernels whose launches are sized to the last byte of 64 KB, or of a share of a compute unit's 160: all their LDS is the launch's.
@pytest.mark.parametrize("family", ["rows_layer_kernel", "panel_layer_kernel", "qgemm_wholek_kernel"])
def test_kernels_sized_by_the_launch_have_no_lds_of_their_own(family):
    sizes = [k[".group_segment_fixed_size"] for k in _kernels() if family in k[".name"]]
    assert sizes and set(sizes) == {0}


def test_num_splits_matches_oracle_everywhere():
    for Cn in list(range(1, 300)) + [512, 1000, 1024, 1500, 2048, 3000, 4096]:
        for r in (0.0, 0.01, 0.02, 0.05, 0.1, 0.2, 0.25, 0.5, 1.0):
            assert B.ocs_num_splits(Cn, r) == ref.num_splits(Cn, r), (Cn, r)
    assert B.ocs_num_splits(0, 0.1) == 0 and B.ocs_num_splits(10, -1.0) == 0


def test_padded_cols_and_workspace():
    assert B.ocs_padded_cols(2358) == 2432
    assert B.ocs_conv_weight_cols(9, 272) == 2496 and B.ocs_conv_weight_cols(0, 16) == 0
    assert B.ocs_padded_channels(262) == 272 and B.ocs_padded_channels(4) == 16
    assert B.ocs_padded_cols(64) == 64 and B.ocs_padded_cols(269) == 272 and B.ocs_padded_cols(68) == 80 and B.ocs_padded_cols(320) == 320 and B.ocs_padded_cols(321) == 384 and B.ocs_padded_cols(0) == 0
    assert B.ocs_workspace_bytes(0, 10) == 0
    for rows, cols in [(1, 1), (64, 256), (12544, 2304), (6000, 3000), (3211264, 147), (802816, 64)]:
        wb = B.ocs_workspace_bytes(rows, cols)
        assert wb >= 4 * cols and wb % 256 == 0
        assert wb < 64 << 20


A = 1 << 20  # a fake, suitably aligned "device address": validation never dereferences it


def _call(fn, *args):
    return getattr(B.lib(), fn)(*args)


def test_argument_errors_are_reported_without_a_device():
    L = B.lib()
    ws = 1 << 24
    # NULL pointers
    assert L.ocs_quantize(None, 4, 4, 4, 8, None, 1.0, A, 64, A, A, ws, None) == -1
    assert L.ocs_split_act(A, 4, 4, 1, 4, None, None, 2, 8, None, 1.0, A, 64, A, A, ws, None) == -1
    assert L.ocs_split_weights(A, 4, 4, 1, 4, 1, 0, None, A, A, None, 0, None, 8, 1.0, None, 0, None, A, ws, None) == -1
    assert L.ocs_split_weights(A, 4, 4, 1, 4, 1, 0, A, A, A, None, 0, None, 8, 1.0, A, 64, None, A, ws, None) == -1
    assert L.ocs_qgemm(A, 64, A, 64, 4, 4, 4, 8, 8, A, A, None, 0, None, 4, None, 0, None) == -1
    assert L.ocs_split_weights_qa(A, 4, 4, 1, 4, 1, A, A, A, None, A, 8, 8, 1.0, A, 64, A, A, ws, None) == -1  # no chan_path
    assert L.ocs_split_weights_qa(A, 4, 4, 1, 4, 1, A, A, A, A, None, 0, 8, 1.0, None, 0, A, A, ws, None) == -1  # no output
    assert L.ocs_split_weights_qa(A, 4, 4, 1, 4, 1, A, A, A, A, A, 4, 8, 1.0, None, 0, A, A, ws, None) == -2    # ldo < (C+s)*g
    assert L.ocs_split_weights_qa(A, 4, 4, 1, 4, 1, A, A, A, A, A, 8, 9, 1.0, None, 0, A, A, ws, None) == -4    # bits
    assert L.ocs_mse_clip_threshold(A, 4, 4, 4, 8, 16, 4, A, None, A, A, ws, None) == -1   # no histogram
    assert L.ocs_mse_clip_threshold(A, 4, 4, 4, 8, 16, 4, A, A, None, A, ws, None) == -1   # no error array
    assert L.ocs_mse_clip_threshold(A, 4, 4, 4, 8, 0, 4, A, A, A, A, ws, None) == -2       # no bins
    assert L.ocs_mse_clip_threshold(A, 4, 4, 4, 8, 9000, 4, A, A, A, A, ws, None) == -2
    assert L.ocs_mse_clip_threshold(A, 4, 4, 4, 1, 16, 4, A, A, A, A, ws, None) == -4
    assert L.ocs_qconv(A, 64, 1, 4, 4, 8, 3, 3, 1, 1, None, 4, 8, 8, A, A, None, 0, A, 4, None) == -1      # no weights
    assert L.ocs_qconv(A, 64, 1, 2, 2, 8, 3, 3, 1, 0, A, 4, 8, 8, A, A, None, 0, A, 4, None) == -2         # kernel larger than image
    assert L.ocs_qconv(A, 72, 1, 4, 4, 8, 3, 3, 1, 1, A, 4, 8, 8, A, A, None, 0, A, 4, None) == -3         # ldc % 16
    assert L.ocs_qconv(A, 64, 1, 4, 4, 80, 3, 3, 1, 1, A, 4, 8, 8, A, A, None, 0, A, 4, None) == -2        # ldc < C_exp
    assert L.ocs_conv_weights_tap_major(A, 4, 8, 9, 64, A, 64, None) == -2                                  # ldq < C_exp*g
    assert L.ocs_qgemm_requant(A, 64, A, 64, 4, 4, 4, 8, 8, A, A, 0, None, 8, None, 0, A, 16, None, None, 0, None) == -1   # no grid
    assert L.ocs_qgemm_requant(A, 64, A, 64, 4, 4, 4, 8, 8, A, A, 0, A, 8, None, 2, A, 16, None, None, 0, None) == -1      # no list
    assert L.ocs_qgemm_requant(A, 64, A, 64, 4, 20, 4, 8, 8, A, A, 0, A, 8, None, 0, A, 16, None, None, 0, None) == -2     # ldyq < N
    assert L.ocs_qgemm_requant(A, 64, A, 64, 4, 4, 4, 8, 8, A, A, 0, A, 8, None, 0, A, 24, None, None, 0, None) == -3      # ldyq % 16
    assert L.ocs_qgemm_requant(A, 64, A, 64, 4, 4, 4, 8, 8, A, A, 0, A, 8, None, 0, A, 16, A, None, 0, None) == -9         # scale_out aliases the grid
    assert L.ocs_fold_weights(A, 64, 4, 4, 1, 2, None, A, 64, A, None) == -1          # split list missing
    assert L.ocs_fold_weights(A, 4, 4, 4, 1, 2, A, A, 64, A, None) == -2             # ldq < (C+s)*g
    assert L.ocs_split_act_qa(A, 4, 4, 1, 4, A, A, A, A, 1, 8, None, A, 64, A, None) == -1     # no threshold
    assert L.ocs_split_act_qa(A, 4, 4, 1, 4, A, A, A, A, 1, 8, A, A, 64, A, None) == -9        # scale_out aliases it
    # shapes
    assert L.ocs_quantize(A, 0, 4, 4, 8, A, 1.0, A, 64, A, A, ws, None) == -2
    assert L.ocs_quantize(A, 4, 8, 4, 8, A, 1.0, A, 64, A, A, ws, None) == -2      # ldx < cols
    assert L.ocs_quantize(A, 4, 100, 100, 8, A, 1.0, A, 64, A, A, ws, None) == -2   # ldq < cols
    assert L.ocs_split_act(A, 4, 4, 0, 4, A, None, 0, 8, A, 1.0, A, 64, A, A, ws, None) == -2
    assert L.ocs_qgemm(A, 64, A, 64, 4, 4, 100, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -2  # ld < Kpad
    assert L.ocs_qgemm(A, 64, A, 64, 4, 8, 4, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -2    # ldy < N
    # a short K: the pitch only has to hold the row in 16-byte pieces; a long K: whole K-steps
    assert L.ocs_qgemm(A, 64, A, 80, 4, 4, 68, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -2   # 64 < 68
    assert L.ocs_qgemm(A, 88, A, 80, 4, 4, 68, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -3   # 88 % 16
    assert L.ocs_qgemm(A, 400, A, 448, 4, 4, 390, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -2  # 400 < 448
    assert L.ocs_qgemm(A, 464, A, 448, 4, 4, 390, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -3  # 464 % 64
    # alignment
    assert L.ocs_quantize(A, 4, 4, 4, 8, A, 1.0, A, 40, A, A, ws, None) == -3
    assert L.ocs_quantize(A, 4, 4, 4, 8, A, 1.0, A + 4, 64, A, A, ws, None) == -3
    assert L.ocs_qgemm(A + 1, 64, A, 64, 4, 4, 4, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -3
    assert L.ocs_quantize(A, 4, 4, 4, 8, None, 1.0, A, 64, A, A + 16, ws, None) == -3   # workspace
    # bits
    for bits in (1, 9, 0, -3):
        assert L.ocs_quantize(A, 4, 4, 4, bits, A, 1.0, A, 64, A, A, ws, None) == -4
    assert L.ocs_qgemm(A, 64, A, 64, 4, 4, 4, 8, 9, A, A, None, 0, A, 4, None, 0, None) == -4
    # splits
    assert L.ocs_split_act(A, 4, 4, 1, 4, A, None, -1, 8, A, 1.0, A, 64, A, A, ws, None) == -5
    assert L.ocs_select_channels(A, 4, 7000, 1, 7000, 1001, A, A, A, None, A, ws, None) == -5
    # overflow: 140000 * 127 * 127 >= 2^31, but fine at 4-bit weights
    ld = 140032
    assert L.ocs_qgemm(A, ld, A, ld, 4, 4, 140000, 8, 8, A, A, None, 0, A, 4, None, 0, None) == -6
    # workspace
    assert L.ocs_quantize(A, 4, 4, 4, 8, None, 1.0, A, 64, A, None, 0, None) == -7
    assert L.ocs_quantize(A, 4, 4, 4, 8, None, 1.0, A, 64, A, A, 16, None) == -7
    assert L.ocs_select_channels(A, 12544, 256, 9, 2304, 6, A, A, A, None, A, 1024, None) == -7
    # mode / key
    assert L.ocs_split_weights(A, 4, 4, 1, 4, 1, 7, A, A, A, None, 0, None, 8, 1.0, None, 0, None, A, ws, None) == -9
    assert L.ocs_tune(b"no_such_key", 1) == -9
    # clip ratio
    for bad in (0.0, -0.5, float("nan"), float("inf")):
        assert L.ocs_quantize(A, 4, 4, 4, 8, None, bad, A, 64, A, A, ws, None) == -10
        assert L.ocs_split_act(A, 4, 4, 1, 4, A, None, 1, 8, None, bad, A, 64, A, A, ws, None) == -10
        assert L.ocs_act_threshold(A, 4, 4, 1, 4, A, None, 1, 8, bad, A, A, ws, None) == -10
        assert L.ocs_split_weights(A, 4, 4, 1, 4, 1, 0, A, A, A, None, 0, None, 8, bad, A, 64, A, A, ws, None) == -10
        assert L.ocs_split_weights_qa(A, 4, 4, 1, 4, 1, A, A, A, A, A, 8, 8, bad, None, 0, A, A, ws, None) == -10
    assert L.ocs_quantize(A, 0, 4, 4, 8, A, -1.0, A, 64, A, A, ws, None) == -2   # a given threshold: the ratio is unused
    for code in range(-10, 1):
        assert len(L.ocs_strerror(code)) > 1
    assert L.ocs_strerror(-99) == b"unknown error code"


def test_static_scratch_entry_point_checks_arguments_and_size_on_the_host():
    L = B.lib()
    # the same argument checks as ocs_split_act, in the same order
    assert L.ocs_split_act_static(None, 4, 4, 1, 4, None, None, 0, 8, None, 1.0, A, 64, A, None) == -1
    assert L.ocs_split_act_static(A, 4, 4, 0, 4, A, None, 0, 8, A, 1.0, A, 64, A, None) == -2
    assert L.ocs_split_act_static(A, 4, 4, 1, 4, A, None, -1, 8, A, 1.0, A, 64, A, None) == -5
    assert L.ocs_split_act_static(A, 4, 4, 1, 4, A, None, 1, 9, A, 1.0, A, 64, A, None) == -4
    assert L.ocs_split_act_static(A, 4, 4, 1, 4, A, None, 1, 8, None, 0.0, A, 64, A, None) == -10
    # a tensor whose scratch need is beyond the array: refused before any device work
    M, Cn, g = 64, 4000, 256                      # the column maxima alone are 4 MB
    assert B.ocs_workspace_bytes(M, Cn * g) > B.STATIC_SCRATCH_BYTES
    assert L.ocs_split_act_static(A, M, Cn, g, Cn * g, None, None, 0, 8, None, 1.0, A, Cn * g, A, None) == -7
    assert L.ocs_split_act_static(A, M, Cn, g, Cn * g, None, None, 0, 8, A, 1.0, A, Cn * g, A, None) == -7
    # every layer shape of the five workloads fits
    from paper_1901_09504_amd import workloads as wl
    for cfg in range(1, 6):
        for layer in wl.config(cfg):
            assert B.ocs_workspace_bytes(layer.M, layer.C * layer.g) <= B.STATIC_SCRATCH_BYTES, layer


def test_split_k_entry_point_checks_shape_and_workspace_on_the_host():
    L = B.lib()
    args = lambda M, N, K, parts, ws, wb: (A, 4864, A, 4864, M, N, K, 8, 8, A, A, None, 0, A, N, parts, ws, wb, None)
    assert B.ocs_qgemm_split_k_workspace_bytes(12544, 512, 4842, 2) == 49 * 2 * 2 * 256 * 256 * 4
    assert B.ocs_qgemm_split_k_workspace_bytes(12544, 512, 4842, 1) == 0        # nothing to split
    assert B.ocs_qgemm_split_k_workspace_bytes(50176, 512, 4842, 2) == 0        # 392 tiles: no counter slot that large
    assert B.ocs_qgemm_split_k_workspace_bytes(256, 256, 128, 3) == 0           # two K-steps, three parts
    assert L.ocs_qgemm_split_k(*args(12544, 512, 4842, 1, A, 1 << 30)) == -2
    assert L.ocs_qgemm_split_k(*args(50176, 512, 4842, 2, A, 1 << 30)) == -2
    assert L.ocs_qgemm_split_k(*args(12544, 512, 4842, 2, None, 0)) == -7
    assert L.ocs_qgemm_split_k(*args(12544, 512, 4842, 2, A, 1000)) == -7
    assert L.ocs_qgemm_split_k(*args(12544, 512, 4842, 2, A + 8, 1 << 30)) == -3
    # the split walks whole K-steps: the tight pitch ocs_qgemm takes for a short K is refused
    short = lambda ld: (A, ld, A, ld, 256, 256, 269, 8, 8, A, A, None, 0, A, 256, 2, A, 1 << 30, None)
    assert L.ocs_qgemm_split_k(*short(272)) == -2
    assert L.ocs_qgemm_split_k(*short(336)) == -3


def test_one_launch_entry_point_says_what_it_serves_and_checks_on_the_host():
    L = B.lib()
    assert B.ocs_split_act_qgemm_fits(802816, 64, 9, 4, 64, 576) and B.ocs_split_act_qgemm_pays(802816, 64, 9, 4, 64, 576)
    assert B.ocs_split_act_qgemm_fits(802816, 64, 1, 4, 256, 64) and not B.ocs_split_act_qgemm_pays(802816, 64, 1, 4, 256, 64)
    assert B.ocs_split_act_qgemm_fits(3211264, 3, 49, 1, 64, 147)          # 147 columns: two whole K-steps and a rest
    assert not B.ocs_split_act_qgemm_fits(100, 3, 9, 1, 64, 27)            # less than one K-step
    assert not B.ocs_split_act_qgemm_fits(12544, 512, 9, 26, 512, 4608)    # more than one tile of output columns
    assert not B.ocs_split_act_qgemm_fits(100, 64, 256, 4, 64, 16384)      # 16384 columns
    assert not B.ocs_split_act_qgemm_fits(100, 64, 64, 40, 64, 4096)       # 2560 appended columns
    call = lambda **k: L.ocs_split_act_qgemm(*[k.get(n, d) for n, d in (
        ("X", A), ("M", 128), ("C", 64), ("g", 1), ("ldx", 64), ("cs", A), ("s", 4), ("bx", 8), ("thr", A), ("Wq", A),
        ("ldw", 80), ("N", 64), ("bw", 8), ("sw", A), ("sxo", None), ("acc", None), ("ldacc", 0), ("Y", A), ("ldy", 64),
        ("stream", None))])
    assert call(X=None) == -1 and call(thr=None) == -1 and call(Wq=None) == -1 and call(Y=None) == -1 and call(cs=None) == -1
    assert call(ldx=60) == -2 and call(ldy=63) == -2 and call(ldw=64) == -2 and call(acc=A, ldacc=8) == -2
    assert call(N=300, ldy=300) == -2 and call(C=3, g=9, ldx=27, s=1, ldw=48) == -2     # not served
    assert call(ldw=88) == -3 and call(Wq=A + 4) == -3
    assert call(bx=9) == -4 and call(s=-1) == -5
    assert call(sxo=A, thr=A) == -9


@pytest.mark.parametrize("C,g,s,N,below,from_", [
    (64, 1, 4, 64, (1, 802816), ()), (127, 1, 4, 256, (1, 802816), ()),               # too narrow at any size
    (128, 1, 4, 128, (), (1, 802816)), (447, 1, 4, 64, (), (1, 802816)),              # ahead at any size
    (448, 1, 4, 128, (1, 64 * 256 - 1), (64 * 256, 802816)), (767, 1, 4, 64, (64 * 256 - 1,), (64 * 256,)),
    (256, 3, 4, 128, (1000, 128 * 256 - 1), (128 * 256,)), (1024, 1, 52, 64, (128 * 256 - 1,), (128 * 256,)),
    (256, 1, 13, 129, (64 * 256 + 1, 802816), (1, 64 * 256)), (128, 1, 4, 256, (64 * 256 + 1,), (64 * 256,)),
    (257, 1, 4, 129, (1, 156 * 256 - 1), (156 * 256, 802816)), (256, 9, 13, 256, (1000, 156 * 256 - 1), (156 * 256,))])
def test_one_launch_pays_by_rows_columns_and_outputs(C, g, s, N, below, from_):
    """Few long rows leave most compute units without a tile: there the two launches are ahead, up to four times
    (rows per compute unit, of which there are 256)."""
    for M in below:
        assert B.ocs_split_act_qgemm_fits(M, C, g, s, N, C * g) and not B.ocs_split_act_qgemm_pays(M, C, g, s, N, C * g)
    for M in from_:
        assert B.ocs_split_act_qgemm_pays(M, C, g, s, N, C * g)


# 256 compute units.  Values of X in a row of tiles, a copy counted twice: up to 27648 (22528 with tiles of 128 columns) launched by
# the host, 13312 (10240) in a captured graph; rows of up to 6144 (4096) values; up to 1024 columns past the whole steps.
@pytest.mark.parametrize("M,C,g,s,N,eager,captured", [
    (64, 256, 1, 13, 256, 1, 1), (1, 3000, 1, 150, 6000, 1, 1), (700, 256, 1, 13, 256, 1, 1), (1000, 3, 49, 1, 64, 1, 1),
    (32, 416, 1, 0, 64, 1, 1), (32, 417, 1, 0, 64, 1, 0), (32, 864, 1, 0, 64, 1, 0), (32, 865, 1, 0, 64, 0, 0),
    (64, 832, 1, 16, 64, 1, 0), (64, 832, 1, 17, 64, 0, 0), (27, 1024, 1, 0, 64, 1, 0), (28, 1024, 1, 0, 64, 0, 0),
    (2, 4096, 1, 0, 64, 1, 1), (2, 4097, 1, 0, 64, 1, 0), (1, 682, 9, 0, 64, 1, 0), (1, 683, 9, 0, 64, 0, 0),
    (1, 1024, 1, 1024, 64, 1, 1), (1, 1024, 1, 1025, 64, 0, 0), (1, 63, 1, 962, 64, 0, 0), (1, 63, 1, 961, 64, 1, 1),
    (700, 320, 1, 0, 1000, 1, 1), (700, 321, 1, 0, 1000, 1, 0), (700, 704, 1, 0, 1000, 1, 0), (700, 705, 1, 0, 1000, 0, 0),
    (20, 3000, 1, 150, 6000, 0, 0), (32, 1000, 1, 50, 64, 0, 0), (8200, 64, 1, 3, 300, 0, 0)])
def test_forward_of_few_tiles_by_what_a_row_of_tiles_holds(M, C, g, s, N, eager, captured):
    ld = B.ocs_padded_cols((C + s) * g)
    assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, False) == eager
    assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, True) == captured


# Rows per compute unit (98 to 128, or from 192 on), whole steps and lines, few copies, rows that follow each other, alignment of X.
@pytest.mark.parametrize("C,g,s,N,extra,inside,outside", [
    (512, 1, 26, 64, 0, (98 * 256, 25088 + 7, 128 * 256, 192 * 256, 802816), (96 * 256, 98 * 256 - 1, 128 * 256 + 1, 160 * 256, 192 * 256 - 1)),
    (256, 9, 12, 256, 0, (98 * 256, 128 * 256, 200704), (97 * 256, 176 * 256)), (512, 9, 25, 1, 0, (98 * 256,), (97 * 256,)),
    (384, 1, 76, 100, 0, (100 * 256,), ()), (384, 1, 77, 100, 0, (), (100 * 256,)), (1024, 1, 204, 64, 0, (200 * 256,), ()),
    (1024, 1, 205, 64, 0, (), (200 * 256,)), (512, 1, 26, 64, 32, (), (100 * 256,)), (1024, 1, 51, 64, 32, (100 * 256,), ()),
    (1024, 1, 51, 64, 8, (), (100 * 256,)), (320, 1, 16, 64, 0, (), (100 * 256, 802816)), (400, 1, 20, 64, 0, (), (100 * 256,)),
    (512, 1, 26, 257, 0, (), (100 * 256,))])
def test_forward_of_many_rows_by_rows_and_copies(C, g, s, N, extra, inside, outside):
    ld = B.ocs_padded_cols((C + s) * g)
    for M in inside:
        assert B.ocs_forward_one_launch(M, C, g, C * g + extra, s, ld, ld, N, X=1 << 20) == 2, M
        assert B.ocs_forward_one_launch(M, C, g, C * g + extra, s, ld, ld, N, captured=True, X=1 << 20) == 2, M
        assert B.ocs_forward_one_launch(M, C, g, C * g + extra, s, ld, ld, N, X=(1 << 20) + 64) == 0, M
    for M in outside:
        assert B.ocs_forward_one_launch(M, C, g, C * g + extra, s, ld, ld, N, X=1 << 20) == 0, M


# One round of 64-row tiles: 44 to 64 rows per compute unit, from 36 on up to 640 columns, from 52 on beyond 2304 with more than 128 outputs;
# whole lines, few copies.
@pytest.mark.parametrize("C,g,s,N,inside,outside", [
    (640, 1, 32, 64, (36 * 256, 64 * 256), (36 * 256 - 1, 64 * 256 + 1)), (704, 1, 35, 256, (44 * 256, 64 * 256), (44 * 256 - 1, 64 * 256 + 1)),
    (256, 9, 6, 256, (12544,), ()), (512, 9, 26, 100, (12544,), ()), (512, 9, 26, 129, (52 * 256, 64 * 256), (52 * 256 - 1, 12544)), (512, 9, 26, 128, (44 * 256,), ()), (512, 9, 26, 257, (), (12544,)), (400, 1, 20, 64, (), (12544,)),
    (320, 1, 16, 64, (), (12544,)), (512, 1, 103, 64, (), (12544,))])
def test_forward_of_one_round_of_64_rows(C, g, s, N, inside, outside):
    ld = B.ocs_padded_cols((C + s) * g)
    for M in inside:
        for captured in (False, True):
            assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, captured=captured, X=1 << 20) == 2, M
        assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, X=(1 << 20) + 64) == 0, M
    for M in outside:
        assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, X=1 << 20) == 0, M


# Rows (more than the layer of few tiles takes: sixteen per compute unit with 256 outputs, 32 with 64), code rows of up to 320 bytes
# (192, and at most 160 columns of X, with more than 128 outputs),
# outputs, more than 2^26 of them in more than 128 columns, padding past the last step; strides and alignment of X do not count.
@pytest.mark.parametrize("C,g,s,N,inside,outside", [
    (3, 49, 1, 64, (32 * 256 + 1, 401408, 3211264), (32 * 256,)), (304, 1, 16, 128, (8200, 802816), (32 * 256,)), (304, 1, 17, 128, (), (8200, 802816)),
    (160, 1, 8, 129, (8200,), ()), (161, 1, 8, 129, (), (8200,)), (150, 1, 50, 129, (), (8200,)), (150, 1, 50, 128, (8200,), ()),
    (64, 1, 4, 256, (16 * 256 + 1, 1 << 18), (16 * 256, (1 << 18) + 1, 802816)), (64, 1, 4, 257, (), (200000,)), (4, 1, 1, 1, (200000,), ()),
    (3, 1, 1, 1, (), (200000,))])
def test_forward_of_short_rows_by_rows_and_outputs(C, g, s, N, inside, outside):
    ld = B.ocs_padded_cols((C + s) * g)
    for M in inside:
        for captured in (False, True):
            assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N, captured=captured) == 3, M
            assert B.ocs_forward_one_launch(M, C, g, C * g + 5, s, ld, ld, N, captured=captured, X=(1 << 20) + 4) == 3, M
        assert B.ocs_forward_one_launch(M, C, g, C * g, s, 384, ld, N) == 0, M
    for M in outside:
        assert B.ocs_forward_one_launch(M, C, g, C * g, s, ld, ld, N) != 3, M


# Where the two launches are ahead among them: few columns at many rows; the start of a second round and an even number of the
# other kernel's tiles with more than 256 columns; more than 128 outputs in whole lines or groups of four with more than 128 code bytes, and in
# a graph with few rows.
@pytest.mark.parametrize("C,s,N,rows,eager,captured", [
    (23, 2, 64, 784 * 256, 3, 3), (23, 2, 64, 784 * 256 + 1, 0, 0), (24, 2, 64, 784 * 256 + 1, 3, 3), (24, 2, 64, 2200 * 256, 3, 3), (63, 4, 64, 2200 * 256 + 1, 0, 0),
    (64, 4, 64, 2200 * 256 + 1, 3, 3), (257, 13, 64, 128 * 256, 3, 3), (257, 13, 64, 128 * 256 + 1, 0, 0), (257, 13, 64, 150 * 256 + 1, 3, 3),
    (257, 13, 65, 140 * 256, 3, 3), (256, 13, 64, 140 * 256, 3, 3), (300, 15, 128, 128 * 256 + 1, 0, 0), (300, 15, 128, 134 * 256 + 1, 3, 3), (300, 15, 128, 190 * 256, 3, 3),
    (300, 15, 128, 190 * 256 + 1, 0, 0), (300, 15, 100, 215 * 256 + 1, 3, 3), (300, 15, 128, 225 * 256, 0, 0), (300, 15, 128, 225 * 256 + 1, 3, 3), (300, 15, 64, 270 * 256, 0, 0),
    (300, 15, 64, 270 * 256 + 1, 3, 3), (300, 15, 50, 215 * 256 + 1, 3, 3),
    (256, 13, 128, 206 * 256, 0, 0), (256, 13, 128, 206 * 256 + 1, 3, 3), (240, 12, 128, 200 * 256, 3, 3), (128, 7, 160, 128 * 256, 3, 3), (128, 7, 160, 128 * 256 + 1, 0, 0), (128, 7, 160, 500 * 256, 0, 0),
    (128, 7, 164, 128 * 256 + 1, 0, 0), (128, 7, 164, 160 * 256 + 1, 3, 3), (128, 7, 162, 140 * 256, 3, 3), (128, 7, 256, 500 * 256, 3, 3), (120, 6, 160, 500 * 256, 3, 3),
    (128, 7, 160, 48 * 256, 3, 3), (128, 7, 160, 48 * 256 - 1, 3, 0), (120, 6, 160, 32 * 256, 3, 3), (120, 6, 160, 32 * 256 - 1, 3, 0), (48, 3, 160, 17 * 256, 3, 3),
    (64, 4, 160, 17 * 256, 3, 0), (64, 4, 196, 17 * 256, 3, 3), (65, 4, 196, 17 * 256, 3, 0), (64, 4, 201, 23 * 256, 3, 0), (64, 4, 201, 24 * 256, 3, 3),
    (128, 7, 201, 23 * 256, 0, 0), (128, 7, 201, 24 * 256, 3, 3)])
def test_forward_of_short_rows_where_two_launches_are_ahead(C, s, N, rows, eager, captured):
    ld = B.ocs_padded_cols(C + s)
    assert B.ocs_forward_one_launch(rows, C, 1, C, s, ld, ld, N, captured=False) == eager
    assert B.ocs_forward_one_launch(rows, C, 1, C, s, ld, ld, N, captured=True) == captured


def test_forward_route_of_refused_shapes_and_forced_kernels():
    assert B.ocs_forward_one_launch(0, 64, 1, 64, 1, 128, 128, 64) == 0 and B.ocs_forward_one_launch(4, 64, 1, 63, 1, 128, 128, 64) == 0
    assert B.ocs_forward_one_launch(4, 64, 1, 64, -1, 128, 128, 64) == 0 and B.ocs_forward_one_launch(4, 64, 1, 64, 1, 128, 128, 0) == 0
    assert B.ocs_forward_one_launch(4, 64, 1, 64, 1, 128, 128, 64) == 1
    for key, value in (("gemm_tile", 7), ("act_grid", 8), ("slice_layer", 0)):
        B.ocs_tune(key, value)
        try:
            assert B.ocs_forward_one_launch(4, 64, 1, 64, 1, 128, 128, 64) == 0, key
        finally:
            B.ocs_tune(key, -1)


def test_binding_raises_on_error():
    with pytest.raises(B.OcsError) as e:
        B._check(-4, "ocs_quantize")
    assert "2..8" in str(e.value) and e.value.code == -4


def test_forward_reports_what_its_two_steps_report():
    L = B.lib()
    ws = 1 << 24

    def fwd(X=A, M=4, C=8, g=1, ldx=8, src=A, s=2, bx=8, thr=A, clip=1.0, Xq=A, ldq=16, sx=A, Wq=A, ldw=16, N=4, bw=8, sw=A,
            acc=None, ldacc=0, Y=A, ldy=4, w=A, wb=ws):
        return L.ocs_forward(X, M, C, g, ldx, src, s, bx, thr, clip, Xq, ldq, sx, Wq, ldw, N, bw, sw, acc, ldacc, Y, ldy, w, wb, None)

    for name in ("X", "src", "Xq", "sx", "Wq", "sw", "Y"):
        assert fwd(**{name: None}) == -1, name
    assert fwd(M=0) == -2 and fwd(ldx=7) == -2 and fwd(N=0) == -2 and fwd(ldq=0) == -2 and fwd(ldy=3) == -2
    assert fwd(ldw=0) == -2 and fwd(acc=A, ldacc=3) == -2
    assert fwd(Xq=A + 1) == -3 and fwd(ldq=24) == -3 and fwd(Wq=A + 4) == -3 and fwd(thr=None, w=A + 16) == -3
    assert fwd(bx=9) == -4 and fwd(bw=1) == -4 and fwd(s=-1) == -5
    assert fwd(C=7000, ldx=140000, g=20, s=0, ldq=140032, ldw=140032) == -6
    assert fwd(thr=None, w=None, wb=0) == -7 and fwd(thr=None, clip=0.0) == -10


def test_first_layer_of_a_chain_reports_what_its_steps_report():
    L = B.lib()

    def fwd(X=A, Bn=1, H=4, W=4, C=8, src=A, s=2, bx=8, thr=A, clip=1.0, Aq=A, ldc=16, sx=A, k=1, stride=1, pad=0, Wt=A, N=4, bw=8, sw=A,
            nt=A, nb=8, ns=A, nn=1, Yq=A, ldyq=16, nso=A + 64, acc=None, ldacc=0, w=A, wb=1 << 24):
        return L.ocs_conv_forward_requant(X, Bn, H, W, C, src, s, bx, thr, clip, Aq, ldc, sx, k, k, stride, pad, Wt, N, bw, sw, 1, nt, nb,
                                          ns, nn, Yq, ldyq, nso, acc, ldacc, w, wb, None)

    for name in ("X", "src", "Aq", "sx", "Wt", "sw", "nt", "ns", "Yq"):
        assert fwd(**{name: None}) == -1, name
    assert fwd(Bn=0) == -2 and fwd(H=0) == -2 and fwd(N=0) == -2 and fwd(ldc=0) == -2 and fwd(k=7) == -2 and fwd(pad=-1) == -2
    assert fwd(stride=0) == -2 and fwd(ldyq=0) == -2 and fwd(acc=A, ldacc=3) == -2
    assert fwd(Aq=A + 1) == -3 and fwd(Wt=A + 4) == -3 and fwd(Yq=A + 4) == -3 and fwd(ldyq=24) == -3 and fwd(thr=None, w=A + 16) == -3
    assert fwd(bx=9) == -4 and fwd(bw=1) == -4 and fwd(nb=9) == -4 and fwd(s=-1) == -5 and fwd(nn=513, ldyq=528) == -5
    assert fwd(thr=None, w=None, wb=0) == -7 and fwd(thr=None, clip=0.0) == -10 and fwd(nso=A) == -9


def test_forward_act_reports_what_its_steps_report():
    L = B.lib()

    def fwd(X=A, M=4, C=8, g=1, ldx=8, s=2, bx=8, clip=1.0, ss=A, cs=A, cd=A, mx=A + 4096, Xq=A, ldq=64, sx=A, Wq=A, ldw=64, N=4, bw=8,
            sw=A, acc=None, ldacc=0, Y=A, ldy=4, w=A, wb=1 << 24):
        return L.ocs_forward_act(X, M, C, g, ldx, s, bx, clip, ss, cs, cd, mx, Xq, ldq, sx, Wq, ldw, N, bw, sw, acc, ldacc, Y, ldy, w, wb,
                                 None)

    for name in ("X", "ss", "cs", "cd", "mx", "Xq", "sx", "Wq", "sw", "Y"):
        assert fwd(**{name: None}) == -1, name
    assert fwd(M=0) == -2 and fwd(ldx=7) == -2 and fwd(N=0) == -2 and fwd(ldq=0) == -2 and fwd(ldw=0) == -2 and fwd(ldy=3) == -2
    assert fwd(acc=A, ldacc=3) == -2
    assert fwd(Xq=A + 1) == -3 and fwd(ldq=24) == -3 and fwd(Wq=A + 4) == -3 and fwd(w=A + 16) == -3
    assert fwd(bx=9) == -4 and fwd(bw=1) == -4 and fwd(s=-1) == -5
    assert fwd(C=7000, ldx=140000, g=20, s=0, ldq=140032, ldw=140032) == -6
    assert fwd(w=None, wb=0) == -7 and fwd(wb=16) == -7
    assert fwd(clip=0.0) == -10 and fwd(clip=-1.0) == -10 and fwd(clip=float("inf")) == -10
    assert fwd(mx=A) == -9 and fwd(mx=A + 4) == -9          # the maximum in scale_x_out: read by one workgroup, written by another
