"""Which kernel the dispatcher takes where two or more cover a layer, on the CPU:
layers measured with each of them (us in the comments, MI355X), on both sides of
the line and a few percent or more apart."""
import os
import re

import numpy as np
import pytest

import paper_1911_08076_amd as P

I8, U2, I32, B64 = (P.IFQ_LAYOUT_I8_NHWC, P.IFQ_LAYOUT_U2_NHWC_PACKED, P.IFQ_LAYOUT_I32_NHWC,
                    P.IFQ_LAYOUT_U2_BLOCK64)


def name(n, h, w, cin, cout, k, stride, in_bits, out_bits, il, ol):
    return P.ifq_conv_kernel_name(
        P.conv_desc(n, h, w, cin, cout, k, stride, k // 2, in_bits, out_bits, il, ol))


@pytest.mark.parametrize("layer,kernel", [
    # general and windowed kernel on byte and packed codes: 14.7 and 23.9 us
    ((23, 165, 164, 48, 32, 3, 2, 2, 2, I8, I8), "conv_igemm<32,"),
    ((3, 91, 89, 48, 32, 1, 1, 2, 2, U2, U2), "conv_igemm<32,"),         # 4.5, 6.1
    ((4, 120, 109, 32, 16, 1, 1, 2, 0, U2, I32), "conv_igemm<16,"),      # 4.5, 5.9
    ((54, 24, 23, 32, 32, 1, 1, 3, 0, I8, I32), "conv_igemm<32,"),       # 4.4, 5.7
    ((8, 168, 149, 160, 32, 1, 1, 2, 0, U2, I32), "conv_igemm<32,"),     # 15.3, 19.1
    ((17, 57, 45, 32, 48, 1, 1, 4, 0, I8, I32), "conv_igemm<64,"),       # 6.4, 7.7
    ((22, 92, 90, 176, 16, 3, 2, 3, 3, I8, I8), "conv_igemm<16,"),       # 30.5, 36.7
    ((32, 27, 27, 96, 256, 5, 1, 4, 4, I8, I8), "conv_win<0,"),          # 67.9, 30
    ((8, 7, 7, 512, 512, 3, 1, 2, 2, I8, I8), "conv_win<0,"),            # 57.7, 7.9
    ((8, 56, 56, 64, 64, 3, 1, 2, 2, I8, I8), "conv_win<0,"),            # 9.9, 7.0
    ((32, 27, 27, 96, 256, 5, 1, 2, 2, U2, U2), "conv_win<1,"),          # 35.4, 26.3
])
def test_general_or_windowed_kernel(layer, kernel):
    assert name(*layer).startswith(kernel), name(*layer)


def join_name(n, h, w, cin, cout, stride, join):
    d = P.conv_desc(n, h, w, cin, cout, 3, stride, 1, 2, 2, B64, B64)
    return P.ifq_conv_kernel_name(d, join)


@pytest.mark.parametrize("layer,kernel", [
    # tiled and windowed kernel on layers of few stages: 8.0 and 9.1 us
    ((16, 28, 28, 128, 512, 1, 1, 2, 2, B64, B64), "conv_mfma<1, 8, 1, 2, 2,"),
    ((8, 56, 56, 64, 256, 1, 1, 2, 2, B64, B64), "conv_mfma<1, 8, 1, 2, 2,"),    # 8.0, 9.2
    ((1, 165, 152, 256, 256, 1, 1, 2, 2, B64, B64), "conv_mfma<1, 8, 1, 2, 2,"), # 9.7, 10.4
    ((2, 69, 67, 64, 320, 1, 1, 2, 0, B64, I32), "conv_mfma<2, 4, 1, 1, 2,"),    # 6.7, 9.3
    ((1, 169, 158, 64, 256, 1, 1, 2, 2, B64, B64), "conv_mfma<1, 8, 1, 2, 2,"),  # 8.2, 9.3
    # and deeper K: 18.9, 10.5
    ((4, 27, 27, 128, 256, 5, 1, 2, 2, B64, B64), "conv_win<2,"),
    ((6, 75, 57, 128, 160, 3, 2, 2, 2, U2, U2), "conv_win<2,"),                  # 12.2, 8.7
    # 3x3 layers on BLOCK64 codes, register-blocked and windowed kernel: 11.1, 8.3
    ((1, 13, 13, 512, 512, 3, 1, 2, 2, B64, B64), "conv_win<2,"),
    ((2, 14, 14, 256, 512, 3, 2, 2, 2, B64, B64), "conv_win<2,"),                # 8.3, 6.4
    ((2, 45, 44, 448, 192, 3, 1, 2, 2, B64, B64), "conv_win<2,"),                # 26.0, 11.8
    ((1, 28, 28, 64, 64, 3, 1, 2, 2, B64, B64), "conv_wv<"),                     # 4.9, 5.2
    ((14, 17, 16, 128, 256, 3, 1, 2, 2, B64, B64), "conv_wv<"),                  # 6.8, 7.7
    # outputs that the register-blocked kernels do not write: 12.8 tiled, 6.6
    ((4, 14, 14, 256, 256, 3, 1, 2, 3, B64, I8), "conv_win<2,"),
    ((2, 54, 54, 512, 448, 3, 1, 2, 0, B64, I32), "conv_halo<"),                 # 23.9, 26.4
])
def test_kernels_on_2_bit_codes(layer, kernel):
    assert name(*layer).startswith(kernel), name(*layer)


def test_kernels_with_an_identity_join():
    table = np.zeros(4, np.int32)    # its address only is looked at
    j = P.make_join(P.IFQ_JOIN_IDENTITY, B64, table, None, [0.5, 1.0, 1.5], table=table)
    assert join_name(16, 7, 7, 512, 512, 1, j).startswith("conv_win<2,")      # 12.3 us, 9.8
    assert join_name(4, 14, 14, 256, 256, 1, j).startswith("conv_win<2,")     # 7.6, 6.8
    assert join_name(8, 28, 28, 128, 128, 1, j).startswith("conv_w")          # 7.4, 7.7
    assert not join_name(8, 28, 28, 128, 128, 1, j).startswith("conv_win<")
    # windows too wide for the register-blocked kernels: 35.3, conv_win 43.7
    assert join_name(10, 80, 64, 448, 448, 2, j).startswith("conv_halo<")


CSRC = os.path.join(os.path.dirname(P.__file__), "csrc")


def test_every_windowed_instance_has_a_parity_case():
    # a refit of the predictions must not leave a tile that still runs without a case:
    # the parity cases name every tile of the table with each of the three inputs, and
    # the dispatcher takes each case there
    from test_gpu_win import CASES
    with open(os.path.join(CSRC, "ifq_conv_win.hip")) as f:
        tiles = re.findall(r"^    IFQ_WV\(([\d, ]+)\),", f.read(), re.M)
    assert len(tiles) == 9
    assert {c[13] for c in CASES} == {"%d, %s" % (i, t) for i in range(3) for t in tiles}
    for n_, n, h, w, ci, co, k, st, pad, ib, ob, il, ol, tile in CASES:
        d = P.conv_desc(n, h, w, ci, co, k, st, pad, ib, ob, il, ol)
        assert P.ifq_conv_kernel_name(d) == "conv_win<%s>" % tile, n_


def test_every_tile_of_the_tiled_and_the_general_kernel_has_a_parity_case():
    from test_gpu_conv import TILED
    from test_gpu_igemm import CASES
    with open(os.path.join(CSRC, "ifq_conv_mfma.hip")) as f:
        tiles = set(re.findall(r'"conv_mfma<([\d, ]+)>"', f.read()))
    assert len(tiles) == 6 and {c[12] for c in TILED} == tiles
    for n_, n, h, w, ci, co, k, st, pad, ob, il, ol, tile in TILED:
        d = P.conv_desc(n, h, w, ci, co, k, st, pad, 2, ob, il, ol)
        assert P.ifq_conv_kernel_name(d) == "conv_mfma<%s>" % tile, n_
    with open(os.path.join(CSRC, "ifq_conv.hip")) as f:
        names = set(re.findall(r'"(conv_igemm<[\d, ]+>)"', f.read()))
    assert len(names) == 12 and {c[12] for c in CASES} == names


@pytest.mark.parametrize("layer", [(16, 8, 64, 1024, 480), (10, 19, 64, 1152, 256),
                                   (6, 59, 64, 1152, 128), (5, 39, 39, 1024, 128)])
def test_no_layer_comes_to_need_a_workspace(layer):
    # where the register-blocked kernels take a layer only split over K, another kernel
    # that needs no workspace is faster
    n, h, w, ci, co = layer
    assert P.ifq_conv_workspace_bytes(P.conv_desc(n, h, w, ci, co, 3, 1, 1, 2, 2, B64, U2)) == 0
