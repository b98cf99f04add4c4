"""GPU parity of the general kernel (conv_igemm) on the layers that it keeps beside
the windowed kernel: each of its tiles with each of its gathers, int32 sums and
codes equal to the oracle's bit for bit."""
import zlib

import numpy as np
import pytest

from gpu_util import (I8, U2, I32, gpu_layer, oracle_layer, expect_layout, make_layer,
                      params_for, codes_for)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1911_08076_amd as P
    return P


# (n, h, w, cin, cout, k, stride, pad, in_bits, out_bits, in, out, kernel)
CASES = [
    # gather of 16-byte units of byte codes, where it is predicted faster
    (12, 73, 53, 16, 16, 2, 3, 1, 3, 2, I8, U2, "conv_igemm<16, 256, 1, 0>"),
    (33, 30, 45, 16, 21, 1, 1, 0, 2, 0, I8, I32, "conv_igemm<32, 128, 1, 0>"),
    (22, 18, 77, 32, 52, 1, 1, 1, 2, 1, I8, I8, "conv_igemm<64, 128, 2, 0>"),
    (21, 4, 32, 320, 109, 2, 3, 2, 2, 3, I8, I8, "conv_igemm<128, 128, 2, 0>"),
    # of 4-byte units of packed codes
    (21, 18, 85, 32, 2, 1, 1, 1, 2, 0, U2, I32, "conv_igemm<16, 256, 1, 1>"),
    (19, 82, 53, 32, 20, 1, 2, 0, 2, 2, U2, U2, "conv_igemm<32, 128, 1, 1>"),
    (31, 13, 77, 32, 44, 1, 1, 0, 2, 0, U2, I32, "conv_igemm<64, 128, 2, 1>"),
    (12, 26, 46, 16, 130, 1, 1, 0, 2, 0, U2, I32, "conv_igemm<128, 128, 2, 1>"),
    # rows too wide for the windowed kernel's LDS
    (1, 3, 8200, 16, 68, 3, 1, 1, 2, 2, U2, U2, "conv_igemm<128, 128, 2, 1>"),
    # byte by byte: c_in not a multiple of 16
    (3, 17, 19, 5, 13, 3, 1, 1, 2, 2, I8, I8, "conv_igemm<16, 256, 1, 2>"),
    (2, 11, 13, 7, 30, 3, 2, 1, 4, 4, I8, I8, "conv_igemm<32, 128, 1, 2>"),
    (2, 9, 14, 21, 60, 2, 1, 0, 3, 0, I8, I32, "conv_igemm<64, 128, 2, 2>"),
    (2, 12, 9, 40, 131, 3, 1, 1, 1, 3, I8, I8, "conv_igemm<128, 128, 2, 2>"),
]


@pytest.mark.parametrize("case", CASES, ids=["%dx%dx%dx%d-%d" % c[:5] for c in CASES])
@pytest.mark.parametrize("dump", [True, False], ids=["sums", "codes"])
def test_igemm_bit_exact(P, case, dump):
    n, h, w, cin, cout, k, st, pad, ib, ob, il, ol, kernel = case
    name = "igemm%d_%d_%d" % (h, cin, cout)
    L = make_layer(name, h, w, cin, cout, k, st, pad, ib, ob)
    d = P.conv_desc(n, h, w, cin, cout, k, st, pad, ib, ob, il, ol)
    assert P.ifq_conv_kernel_name(d) == kernel
    seed = zlib.crc32(name.encode()) % 983
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, w, cin), ib)
    want_acc, want = oracle_layer(L, x, p)
    acc, got = gpu_layer(P, L, n, x, p, in_layout=il, out_layout=ol, dump=dump)
    assert not dump or np.array_equal(acc, want_acc)
    assert np.array_equal(got, expect_layout(want, ol) if ob else want)
