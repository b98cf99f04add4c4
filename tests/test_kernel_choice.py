"""Which kernel the dispatcher takes where two or more cover a layer, on the CPU:
layers measured with each of them (us in the comments, MI355X), on both sides of
the line and a few percent or more apart."""
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
