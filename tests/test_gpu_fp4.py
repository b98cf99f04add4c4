"""GPU parity of the fp4 contraction (ifq_conv_forward_fp4): the 3x3 layers
of the ResNet-18 stack with the 2-bit threshold epilogue, on every variant
of the windowed kernel (64, 128, 256 and 512 channels, a stride-2 layer),
must give the oracle's codes bit for bit (the fp32 sums of +-2 x c/2 are
exact integers)."""
import zlib

import numpy as np
import pytest

from gpu_util import (U2, B64, oracle_layer, expect_layout, make_layer, params_for, codes_for,
                      upload_codes, to_dev, device)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1911_08076_amd as P
    return P


def fp4_kernel(name):
    """Whether a kernel name is an fp4 instance (the fp4 template flag)."""
    import paper_1911_08076_amd as P
    return P.kernel_is_fp4(name)


# name, n, h, c_in, c_out, stride, expected variant
FP4 = [
    ("f4_c64_small_batch", 2, 56, 64, 64, 1, "conv_wv<0, true, 73728, 80896>"),
    ("f4_l2", 3, 28, 128, 128, 1, None),
    ("f4_l2_0_s2", 2, 56, 64, 128, 2, None),
    ("f4_l3", 4, 14, 256, 256, 1, "conv_wv<0, true, 73728, 80896>"),
    ("f4_l4", 6, 7, 512, 512, 1, "conv_w2<1, 2, 4, 2, 2, 3, 2, 0, true, 1, 36864>"),
]


@pytest.mark.parametrize("case", FP4, ids=[c[0] for c in FP4])
def test_fp4_conv_bit_exact(P, case):
    import torch
    name, n, h, cin, cout, st, variant = case
    L = make_layer(name, h, h, cin, cout, 3, st, 1, 2, 2)
    seed = zlib.crc32(name.encode()) % 997
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, h, cin), 2)
    _, want = oracle_layer(L, x, p)
    assert len(np.unique(want)) > 1
    thr = P.ifq_fold_thresholds(cout, 2, 2, 9 * cin, p["alpha"], p["beta_in"], p["q_thr"],
                                bias=p["bias"], mean=p["mean"], var=p["var"], gamma=p["gamma"],
                                bn_beta=p["bn_beta"], eps=p["eps"])
    td = to_dev(thr)
    xd = upload_codes(P, x, B64)
    for out_l in (B64, U2):
        d = P.conv_desc(n, h, h, cin, cout, 3, st, 1, 2, 2, B64, out_l)
        kname = P.ifq_conv_fp4_kernel_name(d)
        assert fp4_kernel(kname), kname
        if variant:
            assert kname == variant
        wd = to_dev(P.ifq_pack_weights_fp4(d, p["w"]))
        ho, wo = P.ifq_conv_output_dims(d)
        ob = P.ifq_tensor_bytes(n, ho, wo, cout, out_l)
        y = torch.full((ob,), 0xA5, dtype=torch.uint8, device=device())
        P.ifq_conv_forward_fp4(d, xd, wd, td, y)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        got = (got.reshape(n, cout // 64, ho, wo, 16) if out_l == B64
               else got.reshape(n, ho, wo, cout // 4))
        assert np.array_equal(got, expect_layout(want, out_l)), (name, out_l, kname)


def test_fp4_offered_for_the_64_channel_tiles(P):
    # the full-batch 64-channel layers run the wave-independent persistent
    # kernel (the slice's weights resident in LDS, one workgroup per CU),
    # which has an fp4 instance
    d = P.conv_desc(64, 56, 56, 64, 64, 3, 1, 1, 2, 2, B64, B64)
    assert P.ifq_conv_kernel_name(d) == "conv_wv<0, false, 73728, 80896>"
    assert P.ifq_conv_fp4_kernel_name(d) == "conv_wv<0, true, 36864, 114688>"
    # with a fused pool fp4 is offered where the windowed kernel's int8 tile has an
    # fp4 instance, which its 64-channel one has not
    pd = P.pool_desc(64, 56, 56, 64, 2, 2, P.IFQ_POOL_VALID, 2, B64)
    assert P.ifq_conv_pool_fp4_kernel_name(d, pd) in ("",) or \
        P.ifq_conv_pool_fp4_kernel_name(d, pd).startswith("conv_halo<")


# identity join (the blocks' second convs): name, n, h, channels
FP4_IDJ = [("f4j_l1_small_batch", 2, 56, 64), ("f4j_l2", 3, 28, 128),
           ("f4j_l3", 4, 14, 256), ("f4j_l4", 6, 7, 512)]


def _epilogue_mode(kname):
    """The epilogue mode template argument of a register-blocked 3x3 kernel
    name (1: identity join)."""
    args = kname[kname.index("<") + 1:-1].split(", ")
    return args[{"conv_w2": 7, "conv_wp": 3, "conv_wv": 0}[kname[:kname.index("<")]]]


@pytest.mark.parametrize("case", FP4_IDJ, ids=[c[0] for c in FP4_IDJ])
def test_fp4_identity_join_bit_exact(P, case):
    import torch
    name, n, h, c = case
    L = make_layer(name, h, h, c, c, 3, 1, 1, 2, 2, join=("identity", "x"))
    seed = zlib.crc32(name.encode()) % 997
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, h, c), 2)
    sc = codes_for(seed + 1, (n, h, h, c), 2)
    _, want = oracle_layer(L, x, p, shortcut=sc)
    assert len(np.unique(want)) > 1
    table = to_dev(P.ifq_fold_join_table(p, p["beta_in"], 2, 9 * c, 2, p["q_thr"]))
    scd = upload_codes(P, sc, B64)
    join = P.make_join(P.IFQ_JOIN_IDENTITY, B64, scd, None, p["q_thr"], table=table)
    xd = upload_codes(P, x, B64)
    d = P.conv_desc(n, h, h, c, c, 3, 1, 1, 2, 2, B64, B64)
    kname = P.ifq_conv_fp4_kernel_name(d, join)
    assert fp4_kernel(kname) and _epilogue_mode(kname) == "1", kname
    wd = to_dev(P.ifq_pack_weights_fp4(d, p["w"]))
    ob = P.ifq_tensor_bytes(n, h, h, c, B64)
    y = torch.full((ob,), 0xA5, dtype=torch.uint8, device=device())
    P.ifq_conv_forward_fp4(d, xd, wd, None, y, join=join)
    torch.cuda.synchronize()
    got = y.cpu().numpy().reshape(n, c // 64, h, h, 16)
    assert np.array_equal(got, expect_layout(want, B64)), (name, kname)


# conv2 of a downsampling block with the 1x1/2 downsample inside the kernel
# (IFQ_JOIN_CONV_FUSED), both convs on fp4: the three ResNet-18 shapes at
# small batch, one ragged
FP4_FUSED = [(2, 56, 64, 128), (3, 28, 128, 256), (2, 14, 256, 512), (5, 13, 64, 128)]


@pytest.mark.parametrize("shape", FP4_FUSED, ids=["x".join(map(str, f)) for f in FP4_FUSED])
def test_fp4_fused_downsample_bit_exact(P, shape):
    import torch
    n, hin, cin, cout = shape
    D = make_layer("down", hin, hin, cin, cout, 1, 2, 0, 2, 0)
    ho = (hin - 1) // 2 + 1
    L = make_layer("conv2", ho, ho, cout, cout, 3, 1, 1, join=("conv", "d", "down"))
    pd = params_for(15 + hin, D)
    p = params_for(16 + hin, L)
    xin = codes_for(15 + hin, (n, hin, hin, cin), 2)
    x = codes_for(16 + hin, (n, ho, ho, cout), 2)
    want_d, _ = oracle_layer(D, xin, pd)
    _, want = oracle_layer(L, x, p, shortcut=want_d, down=pd)
    d = P.conv_desc(n, ho, ho, cout, cout, 3, 1, 1, 2, 2, B64, B64)
    dd = P.conv_desc(n, hin, hin, cin, cout, 1, 2, 0, 2, 0, B64, P.IFQ_LAYOUT_I32_NHWC)
    coef = to_dev(P.ifq_fold_join(P.IFQ_JOIN_CONV, p, pd["beta_in"], down=pd))
    w4 = to_dev(P.ifq_pack_weights_fp4(d, p["w"]))
    dw4 = to_dev(P.ifq_pack_weights_fp4(dd, pd["w"]))
    xind = upload_codes(P, xin, B64)
    xd = upload_codes(P, x, B64)
    join = P.make_join(P.IFQ_JOIN_CONV_FUSED, B64, xind, coef, p["q_thr"], down_w=dw4, down=dd)
    kname = P.ifq_conv_fp4_kernel_name(d, join)
    # a fused join instance on fp4: the windowed kernel's (fused flag true)
    # or the register-blocked kernel's (epilogue mode 2)
    assert fp4_kernel(kname) and (kname.endswith(", true, 4, true, true>") or
                                  kname[8:-1].split(", ")[7] == "2"), kname
    ob = P.ifq_tensor_bytes(n, ho, ho, cout, B64)
    y = torch.full((ob,), 0xA5, dtype=torch.uint8, device=device())
    P.ifq_conv_forward_fp4(d, xd, w4, None, y, join=join)
    torch.cuda.synchronize()
    got = y.cpu().numpy().reshape(n, cout // 64, ho, ho, 16)
    assert np.array_equal(got, expect_layout(want, B64)), (shape, kname)


# conv + fused max-pool on the fp4 path (the VGG and YOLO shapes of the
# window-row pools): name, n, h, c_in, c_out
FP4_POOL = [("f4p_vgg_conv4_3", 2, 28, 512, 512), ("f4p_yolo_c5", 2, 26, 128, 256),
            ("f4p_vgg_conv2_2", 1, 112, 128, 128)]


@pytest.mark.parametrize("case", FP4_POOL, ids=[c[0] for c in FP4_POOL])
def test_fp4_conv_pool_bit_exact(P, case):
    import torch
    import oracle
    name, n, h, cin, cout = case
    L = make_layer(name, h, h, cin, cout, 3, 1, 1, 2, 2)
    seed = zlib.crc32(name.encode()) % 997
    p = params_for(seed, L)
    x = codes_for(seed, (n, h, h, cin), 2)
    _, codes = oracle_layer(L, x, p)
    want = oracle.maxpool(codes, 2, 2, "valid")
    thr = to_dev(P.ifq_fold_thresholds(cout, 2, 2, 9 * cin, p["alpha"], p["beta_in"],
                                       p["q_thr"], bias=p["bias"], mean=p["mean"], var=p["var"],
                                       gamma=p["gamma"], bn_beta=p["bn_beta"], eps=p["eps"]))
    d = P.conv_desc(n, h, h, cin, cout, 3, 1, 1, 2, 2, B64, B64)
    pd = P.pool_desc(n, h, h, cout, 2, 2, P.IFQ_POOL_VALID, 2, B64)
    kname = P.ifq_conv_pool_fp4_kernel_name(d, pd)
    assert kname.startswith("conv_w2<") and P.kernel_is_fp4(kname), kname
    w4 = to_dev(P.ifq_pack_weights_fp4(d, p["w"]))
    xd = upload_codes(P, x, B64)
    ob = P.ifq_tensor_bytes(n, h // 2, h // 2, cout, B64)
    y = torch.full((ob,), 0xA5, dtype=torch.uint8, device=device())
    P.ifq_conv_pool_forward_fp4(d, pd, xd, w4, thr, y)
    torch.cuda.synchronize()
    got = y.cpu().numpy().reshape(n, cout // 64, h // 2, h // 2, 16)
    assert np.array_equal(got, expect_layout(want, B64)), (name, kname)
