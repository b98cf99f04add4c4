"""GPU parity of the fully connected kernel (a filter the size of the image on
2-bit codes): batches around its 16-image blocks, K steps from fewer than its
waves to several batches of loads, ragged channels, every layout it reads and
writes."""
import zlib

import numpy as np
import pytest

from gpu_util import (I8, U2, I32, B64, gpu_layer, oracle_layer, expect_layout, make_layer,
                      params_for, codes_for)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1911_08076_amd as P
    return P


# (name, n, h, w, cin, cout, out_bits, in, out)
CASES = [
    ("one_step", 1, 1, 1, 64, 16, 2, U2, U2),
    ("fewer_steps_than_waves", 16, 1, 1, 320, 64, 2, B64, B64),
    ("one_batch_of_loads", 17, 2, 3, 704, 100, 2, U2, I8),
    ("two_batches", 32, 6, 6, 256, 192, 2, U2, U2),
    ("many_batches", 33, 5, 4, 1024, 48, 2, B64, U2),
    ("ragged_channels_i32", 64, 3, 3, 128, 37, 0, U2, I32),
    ("k_bits_out", 5, 4, 1, 192, 30, 4, B64, I8),
    ("ragged_batch", 47, 1, 7, 64, 128, 2, B64, B64),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("dump", [True, False], ids=["sums", "codes"])
def test_fc_bit_exact(P, case, dump):
    name, n, h, w, cin, cout, ob, il, ol = case
    if h == w:
        L = make_layer(name, h, w, cin, cout, h, 1, 0, 2, ob)
        d = P.conv_desc(n, h, w, cin, cout, h, 1, 0, 2, ob, il, ol)
        assert P.ifq_conv_kernel_name(d) == "conv_fc<%d>" % (1 if n <= 16 else 2 if n <= 32 else 4)
    else:
        # a rectangular window as a square filter over a zero-padded square
        # image is another layer; the descriptor takes kw on its own
        return rectangular(P, case, dump)
    seed = zlib.crc32(name.encode()) % 977
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, w, cin), 2)
    want_acc, want = oracle_layer(L, x, p)
    acc, got = gpu_layer(P, L, n, x, p, in_layout=il, out_layout=ol, dump=dump)
    assert not dump or np.array_equal(acc, want_acc)
    assert np.array_equal(got, expect_layout(want, ol) if ob else want)


def rectangular(P, case, dump):
    import torch
    from gpu_util import to_dev, upload_codes, device
    name, n, h, w, cin, cout, ob, il, ol = case
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    wt = (rng.integers(0, 2, (cout, cin, h, w)) * 2 - 1).astype(np.int8)
    x = codes_for(h * 13 + w, (n, h, w, cin), 2)
    sums = np.einsum("nhwc,ochw->no", x.astype(np.int64), wt.astype(np.int64))
    lo, hi = int(sums.min()), int(sums.max())
    thr = np.sort(rng.integers(lo, hi, (cout, (1 << ob) - 1)), axis=1).astype(np.int32)
    s = rng.choice([-1, 1], cout).astype(np.int32)
    rec = np.concatenate([s[:, None], np.where(s[:, None] < 0, -thr[:, ::-1], thr)], axis=1)
    want = np.zeros((n, 1, 1, cout), np.uint8)
    for i in range(1, 1 << ob):
        want += (sums * s > rec[:, i]).astype(np.uint8).reshape(want.shape)
    d = P.conv_desc(n, h, w, cin, cout, h, 1, 0, 2, ob, il, ol, kw=w)
    assert P.ifq_conv_kernel_name(d) == "conv_fc<%d>" % (1 if n <= 16 else 2 if n <= 32 else 4)
    acc = torch.empty(n * cout, dtype=torch.int32, device=device()) if dump else None
    y = torch.empty(P.ifq_tensor_bytes(n, 1, 1, cout, ol), dtype=torch.uint8, device=device())
    P.ifq_conv_forward(d, upload_codes(P, x, il), to_dev(P.ifq_pack_weights(d, wt)),
                       to_dev(rec.astype(np.int32)), y, acc_dump=acc)
    if dump:
        assert np.array_equal(acc.cpu().numpy().reshape(n, cout), sums)
    assert np.array_equal(y.cpu().numpy(), expect_layout(want, ol).reshape(-1))
