"""GPU parity of the windowed kernel for byte codes and 2-bit codes of any
filter size (conv_win): int32 sums and codes equal to the oracle's bit for bit, at the
edges of its tiles, window chunks and epilogues."""
import zlib

import numpy as np
import pytest

import oracle
from gpu_util import (I8, U2, I32, B64, gpu_layer, oracle_layer, expect_layout, make_layer,
                      params_for, codes_for, to_dev, device)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1911_08076_amd as P
    return P


# (name, n, h, w, cin, cout, k, stride, pad, in_bits, out_bits, in, out, template
# arguments of the instance that runs it). Every tile with every kind of input is here.
CASES = [
    ("one_pixel", 1, 1, 1, 16, 80, 1, 1, 0, 2, 2, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("all_padding_taps", 3, 1, 1, 32, 33, 3, 1, 1, 4, 4, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("pad_wider_than_filter", 2, 3, 4, 16, 20, 3, 2, 4, 3, 3, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("stride_past_filter", 2, 13, 11, 48, 40, 2, 3, 0, 2, 2, I8, U2, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("images_per_tile", 37, 3, 3, 64, 64, 3, 1, 1, 2, 2, I8, B64, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("chunks_of_64", 2, 21, 19, 512, 96, 3, 1, 1, 2, 2, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("three_window_buffers", 3, 28, 28, 384, 128, 3, 1, 1, 7, 2, I8, U2, "0, 1, 2, 4, 1, 1, 2, 3"),
    ("one_chunk_odd_units", 2, 9, 8, 304, 24, 3, 1, 1, 5, 1, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("5x5_s1_wide", 3, 57, 61, 96, 144, 5, 1, 2, 4, 4, I8, I8, "0, 1, 4, 2, 1, 2, 2, 3"),
    ("k_split_8", 4, 7, 7, 512, 80, 3, 1, 1, 1, 3, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("1x1_s2_i32", 5, 17, 15, 80, 72, 1, 2, 0, 4, 0, I8, I32, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("even_filter", 2, 10, 12, 32, 16, 4, 2, 1, 2, 4, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("units_past_c_in", 2, 45, 43, 368, 128, 3, 2, 1, 2, 4, I8, I8, "0, 1, 2, 4, 1, 1, 1, 4"),
    ("tile_128x256", 8, 81, 76, 32, 96, 1, 1, 0, 2, 4, I8, I8, "0, 2, 4, 1, 2, 2, 2, 3"),
    ("tile_128x64", 13, 19, 18, 96, 352, 1, 1, 0, 2, 2, I8, U2, "0, 2, 2, 2, 2, 1, 2, 3"),
    ("tile_64x256", 3, 81, 81, 240, 141, 1, 1, 0, 2, 4, I8, I8, "0, 1, 4, 2, 2, 2, 2, 3"),
    ("tile_64x128", 8, 81, 80, 80, 144, 1, 2, 0, 4, 4, I8, I8, "0, 1, 4, 2, 2, 1, 2, 3"),
    ("tile_32x256", 21, 13, 13, 16, 304, 3, 1, 1, 2, 2, I8, I8, "0, 1, 4, 2, 1, 2, 2, 3"),
    ("tile_128x64_4_bits", 3, 45, 44, 160, 237, 1, 1, 0, 4, 4, I8, I8, "0, 2, 2, 2, 2, 1, 2, 3"),
    ("k_split_8_5x5_s2", 3, 9, 8, 368, 304, 5, 2, 2, 2, 4, I8, I8, "0, 1, 1, 8, 1, 1, 1, 3"),
    ("u2_one_unit", 2, 23, 31, 16, 80, 3, 1, 1, 2, 2, U2, U2, "1, 1, 1, 8, 1, 1, 1, 3"),
    ("u2_odd_units", 3, 12, 10, 240, 100, 3, 2, 1, 2, 2, U2, U2, "1, 1, 1, 8, 1, 1, 1, 3"),
    ("u2_5x5", 3, 27, 27, 96, 256, 5, 1, 2, 2, 2, U2, B64, "1, 1, 2, 4, 1, 1, 2, 3"),
    ("u2_k_bits_out", 2, 9, 9, 48, 70, 3, 1, 1, 2, 4, U2, I8, "1, 1, 1, 8, 1, 1, 1, 3"),
    ("u2_i32", 2, 9, 9, 176, 30, 1, 1, 0, 2, 0, U2, I32, "1, 1, 1, 8, 1, 1, 1, 3"),
    ("f_3x3_s2", 6, 75, 57, 128, 160, 3, 2, 1, 2, 2, U2, U2, "2, 1, 4, 2, 2, 1, 2, 3"),
    ("f_images_per_tile", 9, 7, 7, 512, 512, 3, 1, 1, 2, 2, U2, B64, "2, 1, 1, 8, 1, 1, 1, 3"),
    ("f_5x5_blocks", 4, 27, 27, 128, 256, 5, 1, 2, 2, 2, B64, B64, "2, 1, 2, 4, 1, 1, 2, 3"),
    ("f_5x5_s2", 2, 112, 86, 64, 330, 5, 2, 2, 2, 2, B64, I8, "2, 1, 4, 2, 2, 1, 2, 3"),
    ("f_1x1_blocks", 5, 19, 23, 320, 192, 1, 2, 0, 2, 2, B64, U2, "2, 1, 1, 8, 1, 1, 1, 3"),
    ("f_1x1_i32", 8, 16, 12, 256, 193, 1, 1, 0, 2, 0, B64, I32, "2, 1, 2, 4, 1, 1, 1, 4"),
    ("f_wide", 9, 60, 52, 128, 448, 5, 2, 2, 2, 2, B64, B64, "2, 1, 4, 2, 1, 2, 2, 3"),
    ("f_even_filter", 3, 20, 18, 192, 48, 4, 1, 2, 2, 4, U2, I8, "2, 1, 1, 8, 1, 1, 1, 3"),
    ("tile_64x64", 2, 83, 78, 16, 367, 1, 3, 0, 3, 2, I8, I8, "0, 1, 2, 4, 2, 1, 1, 3"),
    ("tile_32x64", 31, 18, 15, 96, 1, 2, 1, 1, 4, 2, I8, I8, "0, 1, 2, 4, 1, 1, 2, 3"),
    ("u2_tile_128x256", 17, 54, 51, 16, 330, 1, 2, 0, 2, 4, U2, I8, "1, 2, 4, 1, 2, 2, 2, 3"),
    ("u2_tile_128x64", 4, 100, 67, 16, 384, 2, 3, 1, 2, 2, U2, I8, "1, 2, 2, 2, 2, 1, 2, 3"),
    ("u2_tile_64x256", 44, 115, 120, 48, 34, 2, 4, 1, 2, 4, U2, I8, "1, 1, 4, 2, 2, 2, 2, 3"),
    ("u2_tile_64x128", 7, 31, 31, 32, 172, 1, 1, 0, 2, 3, U2, I8, "1, 1, 4, 2, 2, 1, 2, 3"),
    ("u2_tile_32x256", 13, 32, 24, 16, 448, 1, 2, 0, 2, 3, U2, I8, "1, 1, 4, 2, 1, 2, 2, 3"),
    ("u2_tile_64x64", 6, 75, 51, 16, 73, 1, 2, 0, 2, 1, U2, I8, "1, 1, 2, 4, 2, 1, 1, 3"),
    ("u2_tile_32x64", 2, 50, 34, 16, 73, 1, 1, 0, 2, 2, U2, I8, "1, 1, 2, 4, 1, 1, 1, 4"),
    ("f_tile_128x256", 47, 21, 19, 64, 197, 1, 1, 0, 2, 2, U2, I8, "2, 2, 4, 1, 2, 2, 2, 3"),
    ("f_tile_128x64", 9, 21, 17, 64, 640, 1, 1, 0, 2, 2, U2, B64, "2, 2, 2, 2, 2, 1, 2, 3"),
    ("f_tile_64x256", 25, 116, 108, 64, 37, 2, 3, 0, 2, 4, U2, I8, "2, 1, 4, 2, 2, 2, 2, 3"),
    ("f_tile_64x64", 6, 23, 17, 64, 197, 1, 1, 0, 2, 2, U2, I8, "2, 1, 2, 4, 2, 1, 1, 3"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("dump", [True, False], ids=["sums", "codes"])
def test_conv_win_bit_exact(P, case, dump):
    name, n, h, w, cin, cout, k, st, pad, ib, ob, il, ol, tile = case
    L = make_layer(name, h, w, cin, cout, k, st, pad, ib, ob)
    d = P.conv_desc(n, h, w, cin, cout, k, st, pad, ib, ob, il, ol)
    assert P.ifq_conv_kernel_name(d) == "conv_win<%s>" % tile
    seed = zlib.crc32(name.encode()) % 983
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, w, cin), ib)
    want_acc, want = oracle_layer(L, x, p)
    acc, got = gpu_layer(P, L, n, x, p, in_layout=il, out_layout=ol, dump=dump)
    assert not dump or np.array_equal(acc, want_acc)
    assert np.array_equal(got, expect_layout(want, ol))


@pytest.mark.parametrize("ob,ol,sl", [(2, I8, I8), (2, U2, U2), (3, I8, I8), (2, B64, B64)])
def test_conv_win_identity_join(P, ob, ol, sl):
    cout = 128 if ol == B64 else 72
    L = make_layer("join", 9, 11, 96, cout, 3, 1, 1, 2, ob, join=("identity", "x"))
    p = params_for(3, L)
    x = codes_for(3, (3, 9, 11, 96), 2)
    sc = codes_for(4, (3, 9, 11, cout), 2)
    want_acc, want = oracle_layer(L, x, p, shortcut=sc)
    acc, got = gpu_layer(P, L, 3, x, p, in_layout=I8, out_layout=ol, shortcut=sc, sc_layout=sl)
    assert np.array_equal(acc, want_acc)
    assert np.array_equal(got, expect_layout(want, ol))


def test_conv_win_identity_join_fragment_order(P):
    L = make_layer("join", 13, 11, 128, 192, 3, 1, 1, 2, 2, join=("identity", "x"))
    p = params_for(13, L)
    x = codes_for(13, (7, 13, 11, 128), 2)
    sc = codes_for(14, (7, 13, 11, 192), 2)
    want_acc, want = oracle_layer(L, x, p, shortcut=sc)
    for sl in (U2, B64, I8):
        acc, got = gpu_layer(P, L, 7, x, p, in_layout=U2, out_layout=U2, shortcut=sc, sc_layout=sl)
        assert np.array_equal(acc, want_acc)
        assert np.array_equal(got, expect_layout(want, U2))


def test_conv_win_conv_join(P):
    L = make_layer("cjoin", 7, 9, 64, 50, 3, 1, 1, 2, 2, join=("conv", "d", "down"))
    D = make_layer("down", 14, 18, 32, 50, 1, 2, 0, 2, 0)
    p, pd = params_for(5, L), params_for(6, D)
    x = codes_for(5, (4, 7, 9, 64), 2)
    dn, _ = oracle_layer(D, codes_for(6, (4, 14, 18, 32), 2), pd)
    want_acc, want = oracle_layer(L, x, p, shortcut=dn, down=pd)
    acc, got = gpu_layer(P, L, 4, x, p, shortcut=dn, down=pd)
    assert np.array_equal(acc, want_acc)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("ob", [1, 2, 4])
def test_conv_win_thresholds_in_any_order(P, ob):
    # records whose thresholds do not ascend, and saturated ones, count the
    # same as any others
    import torch
    n, h, w, cin, cout = 2, 9, 7, 64, 40
    rng = np.random.default_rng(ob)
    d = P.conv_desc(n, h, w, cin, cout, 3, 1, 1, 2, ob)
    assert P.ifq_conv_kernel_name(d).startswith("conv_win<")
    L = make_layer("order", h, w, cin, cout, 3, 1, 1, 2, ob)
    p = params_for(9, L)
    x = codes_for(9, (n, h, w, cin), 2)
    acc = oracle.conv_acc(x, p["w"], 1, 1, 2)
    B = 9 * cin * 3
    thr = rng.integers(-120, 120, (cout, 1 << ob)).astype(np.int32)
    thr[:, 0] = rng.choice([-1, 1], cout)
    thr[0, 1:] = -B - 1
    thr[1, 1:] = B
    want = np.zeros(acc.shape, np.uint8)
    for i in range(1, 1 << ob):
        want += (acc * thr[:, 0] > thr[:, i]).astype(np.uint8)
    y = torch.empty(want.size, dtype=torch.uint8, device=device())
    P.ifq_conv_forward(d, to_dev(x), to_dev(P.ifq_pack_weights(d, p["w"])), to_dev(thr), y)
    assert np.array_equal(y.cpu().numpy().reshape(want.shape), want)


def test_misaligned_input_takes_the_general_kernel(P):
    # conv_win moves 16-byte cells; the same layer from an input that is only
    # 4-byte aligned runs on the general kernel with the same result
    import torch
    n, h, w, cin, cout = 2, 9, 7, 32, 40
    L = make_layer("misaligned", h, w, cin, cout, 3, 1, 1, 4, 4)
    p = params_for(11, L)
    x = codes_for(11, (n, h, w, cin), 4)
    _, want = oracle_layer(L, x, p)
    d = P.conv_desc(n, h, w, cin, cout, 3, 1, 1, 4, 4)
    thr = to_dev(P.ifq_fold_thresholds(cout, 4, 4, 9 * cin, p["alpha"], p["beta_in"], p["q_thr"],
                                       mean=p["mean"], var=p["var"], gamma=p["gamma"],
                                       bn_beta=p["bn_beta"], eps=p["eps"]))
    wd = to_dev(P.ifq_pack_weights(d, p["w"]))
    buf = torch.zeros(x.size + 64, dtype=torch.uint8, device=device())
    y = torch.empty(want.size, dtype=torch.uint8, device=device())
    for off in (0, 4, 16, 20):
        buf[off:off + x.size] = to_dev(x)
        y.zero_()
        P.ifq_conv_forward(d, buf[off:off + x.size], wd, thr, y)
        assert np.array_equal(y.cpu().numpy().reshape(want.shape), want), off


# 3x3 layers on BLOCK64 codes with at most one 32 x 64 tile per CU, up to the
# edge of that rule, ragged tiles and channel blocks
SMALL_B64 = [("sb_13", 1, 13, 13, 512, 512), ("sb_13_b4", 4, 13, 13, 512, 512),
             ("sb_edge", 16, 32, 16, 128, 64), ("sb_odd", 3, 9, 17, 192, 320),
             ("sb_one_px", 1, 1, 1, 128, 64), ("sb_c_out96", 2, 28, 28, 128, 96)]


@pytest.mark.parametrize("case", SMALL_B64, ids=[c[0] for c in SMALL_B64])
def test_conv_win_small_block64(P, case):
    name, n, h, w, cin, cout = case
    L = make_layer(name, h, w, cin, cout, 3, 1, 1, 2, 2)
    p = params_for(21, L)
    x = codes_for(21, (n, h, w, cin), 2)
    want_acc, want = oracle_layer(L, x, p)
    for ol in (B64, U2):
        if ol == B64 and cout % 64:
            continue
        d = P.conv_desc(n, h, w, cin, cout, 3, 1, 1, 2, 2, B64, ol)
        assert P.ifq_conv_kernel_name(d).startswith("conv_win<2,"), P.ifq_conv_kernel_name(d)
        acc, got = gpu_layer(P, L, n, x, p, in_layout=B64, out_layout=ol)
        assert np.array_equal(acc, want_acc)
        assert np.array_equal(got, expect_layout(want, ol))
