"""The LDS-patch kernel's results other than the plain NHWC tensor (NCHW, l_a != 0, odd channel
counts, raw accumulators) against the simple kernel, bit for bit: both evaluate the same
expressions in the same order."""
import numpy as np
import pytest
import torch

from paper_1908_05033_amd import binding as B

pytestmark = pytest.mark.gpu

# N, C_in, H, W, C_out, R, stride, pad
GEOMS = [(2, 24, 7, 9, 33, 3, 1, 1), (1, 130, 13, 11, 130, 3, 2, 1), (3, 64, 1, 1, 66, 3, 1, 2), (2, 70, 9, 6, 259, 1, 2, 0),
         (2, 129, 12, 17, 64, 3, 1, 0)]


def _run(geom, bits, flags, la, layout, with_acc):
    N, C, H, W, K, R, stride, pad = geom
    g = torch.Generator().manual_seed(sum(geom) + bits)
    buf = B.alloc_layer(N, C, H, W, K, R, R, stride, pad, bits, with_acc=with_acc, flags=flags)
    x = torch.randn((N, H, W, C), generator=g).cuda()
    w = torch.randn((K, C, R, R), generator=g).cuda()
    lw, uw = w.reshape(K, -1).amin(1) * 0.9, w.reshape(K, -1).amax(1)
    B.dsq_quantize_act(x, B.DSQ_NHWC, N, C, H, W, la, 2.5, bits, buf.act_packed, buf.pix_code_sum)
    B.dsq_pack_weights(w, lw.contiguous(), uw.contiguous(), None, K, C, R, R, bits, buf.w_packed, buf.w_aux)
    out = torch.full_like(buf.out.reshape(-1), float("nan"))
    acc = torch.full_like(out, -1, dtype=torch.int32) if with_acc else None
    B.dsq_conv2d(buf.desc, buf.act_packed, buf.pix_code_sum, la, 2.5, buf.w_packed, buf.w_aux, out, layout, acc)
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.int32), acc.cpu().numpy() if with_acc else None


@pytest.mark.parametrize("layout", [B.DSQ_NHWC, B.DSQ_NCHW])
@pytest.mark.parametrize("la", [0.0, -2.1, 0.3])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("geom", GEOMS)
def test_same_bits_as_the_simple_kernel(geom, bits, la, layout):
    want = _run(geom, bits, B.DSQ_CONV_KERNEL(1), la, layout, True)
    for kernel in (2, 3, 4, 5, 6):                 # the patch kernel's own choice and its four tiles
        for with_acc in (False, True):
            try:
                got = _run(geom, bits, B.DSQ_CONV_KERNEL(kernel), la, layout, with_acc)
            except B.DsqError as e:
                if e.status != 5 or kernel == 2:   # (a forced tile may not take the layer; its own choice does)
                    raise
                continue
            assert np.array_equal(got[0], want[0]), kernel
            assert not with_acc or np.array_equal(got[1], want[1]), kernel


@pytest.mark.parametrize("layout", [B.DSQ_NHWC, B.DSQ_NCHW])
def test_largest_patch_with_the_tables_of_l_a(layout):
    """The most LDS a launch asks for: a patch near the limit and the tables of l_a != 0 behind it."""
    geom = (300, 512, 1, 3, 300, 3, 2, 2)
    d = B.make_desc(*geom[:5], 3, 3, 2, 2, 2, B.DSQ_CONV_KERNEL(6))
    assert int(B.dsq_conv2d_plan(d, l_a=-2.1).split()[-3]) > 150 * 1024
    want = _run(geom, 2, B.DSQ_CONV_KERNEL(1), -2.1, layout, True)
    got = _run(geom, 2, B.DSQ_CONV_KERNEL(6), -2.1, layout, True)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


# one case per form of the results' epilogue: channel tiles that do not exist, images of one row or
# column (only the middle taps), two rows of padding, two wave groups, 9 classes of borders, and on both
# sides of the rule between the two layouts of a lane (1x1, l_a != 0, a fifth of the channels missing)
@pytest.mark.parametrize("geom", [(2, 64, 5, 8, 96, 3, 1, 1), (1, 512, 7, 7, 97, 3, 1, 1), (2, 40, 1, 9, 36, 3, 1, 1),
                                  (2, 40, 9, 1, 36, 3, 2, 1), (1, 64, 6, 5, 40, 3, 1, 2), (1, 64, 6, 5, 41, 3, 2, 2),
                                  (2, 64, 7, 7, 48, 1, 1, 0), (2, 64, 7, 7, 52, 1, 1, 0), (3, 24, 20, 20, 144, 1, 1, 0),
                                  (3, 30, 33, 17, 31, 1, 2, 0)])
@pytest.mark.parametrize("bits", [1, 3])
def test_nhwc_results_with_an_offset(geom, bits):
    want = _run(geom, bits, B.DSQ_CONV_KERNEL(1), -0.9, B.DSQ_NHWC, False)
    for kernel in (2, 3, 4, 5, 6):
        try:
            got = _run(geom, bits, B.DSQ_CONV_KERNEL(kernel), -0.9, B.DSQ_NHWC, False)
        except B.DsqError as e:
            if e.status != 5 or kernel == 2:
                raise
            continue
        assert np.array_equal(got[0], want[0]), kernel


# two rows of padding: pixels that lack one and two rows or columns of taps, images of one to three rows or
# columns, all of whose pixels do, one and two wave groups, tiles that hold several images
@pytest.mark.parametrize("layout", [B.DSQ_NHWC, B.DSQ_NCHW])
@pytest.mark.parametrize("geom", [(2, 64, 1, 9, 40, 3, 1, 2), (2, 40, 9, 1, 41, 3, 2, 2), (3, 130, 2, 2, 66, 3, 1, 2),
                                  (3, 64, 3, 2, 96, 3, 2, 2), (2, 257, 13, 10, 130, 3, 1, 2), (5, 24, 28, 30, 70, 3, 1, 2)])
@pytest.mark.parametrize("bits", [1, 3])
def test_two_rows_of_padding(geom, bits, layout):
    test_same_bits_as_the_simple_kernel(geom, bits, 0.7, layout)
