"""The split-K kernel for layers of few output tiles against the simple kernel, bit for bit: both add the same
exact integers and evaluate the same expressions in the same order."""
import numpy as np
import pytest
import torch

from paper_1908_05033_amd import binding as B

pytestmark = pytest.mark.gpu

# N, C_in, H, W, C_out, R, stride, pad: pixels and channels past the tiles' ends, waves without a step, one
# to nine steps a wave and more than are in flight together, borders on every side, images inside a tile
GEOMS = [(1, 64, 1, 1, 1, 1, 1, 0), (3, 130, 7, 5, 33, 1, 2, 0), (1, 300, 6, 6, 70, 1, 1, 0), (2, 24, 7, 9, 34, 3, 1, 1),
         (1, 130, 13, 11, 132, 3, 2, 1), (3, 64, 1, 2, 66, 3, 1, 2), (2, 257, 9, 8, 96, 3, 1, 0), (1, 700, 7, 7, 40, 3, 1, 1),
         (1, 64, 61, 67, 64, 3, 1, 1), (2, 128, 56, 56, 128, 3, 2, 1)]


def _prepare(geom, bits, la):
    N, C, H, W, K, R, stride, pad = geom
    g = torch.Generator().manual_seed(sum(geom) + bits)
    buf = B.alloc_layer(N, C, H, W, K, R, R, stride, pad, bits, with_acc=True)
    x = torch.randn((N, H, W, C), generator=g).cuda()
    w = torch.randn((K, C, R, R), generator=g).cuda()
    lw, uw = w.reshape(K, -1).amin(1) * 0.9, w.reshape(K, -1).amax(1) + 0.1
    B.dsq_quantize_act(x, B.DSQ_NHWC, N, C, H, W, la, 2.5, bits, buf.act_packed, buf.pix_code_sum)
    B.dsq_pack_weights(w, lw.contiguous(), uw.contiguous(), None, K, C, R, R, bits, buf.w_packed, buf.w_aux)
    return buf


def _desc(geom, bits, flags):
    N, C, H, W, K, R, stride, pad = geom
    return B.make_desc(N, C, H, W, K, R, R, stride, pad, bits, flags)


@pytest.mark.parametrize("layout", [B.DSQ_NHWC, B.DSQ_NCHW])
@pytest.mark.parametrize("la", [0.0, -2.1])
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("geom", GEOMS)
def test_same_bits_as_the_simple_kernel(geom, bits, la, layout):
    buf = _prepare(geom, bits, la)
    assert B.dsq_conv2d_plan(_desc(geom, bits, 0), l_a=la).startswith("split-K kernel for few output tiles")
    got = []
    for kernel, with_acc in ((1, True), (0, True), (0, False)):
        out = torch.full_like(buf.out.reshape(-1), float("nan"))
        acc = torch.full_like(out, -1, dtype=torch.int32) if with_acc else None
        B.dsq_conv2d(_desc(geom, bits, B.DSQ_CONV_KERNEL(kernel)), buf.act_packed, buf.pix_code_sum, la, 2.5, buf.w_packed, buf.w_aux,
                     out, layout, acc)
        got.append((out.cpu().numpy().view(np.int32), acc.cpu().numpy() if with_acc else None))
    assert np.array_equal(got[1][0], got[0][0]) and np.array_equal(got[1][1], got[0][1])
    assert np.array_equal(got[2][0], got[0][0])


@pytest.mark.parametrize("affine", [False, True])
@pytest.mark.parametrize("la", [0.0, -2.1])
@pytest.mark.parametrize("bits,bits_next,dense", [(2, 2, False), (4, 4, False), (4, 3, True), (1, 4, False)])
@pytest.mark.parametrize("geom", [g for g in GEOMS if g[4] > 64 or g[1] == 700])
def test_chained_same_codes_as_the_simple_kernel(geom, bits, bits_next, dense, la, affine):
    N, C, H, W, K, R, stride, pad = geom
    buf = _prepare(geom, bits, la)
    next_flag = B.DSQ_CONV_NEXT_DENSE3 if dense else 0
    assert B.dsq_conv2d_plan(_desc(geom, bits, next_flag), chained=True, l_a=la).startswith("split-K kernel for few output tiles")
    Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    g = torch.Generator().manual_seed(7)
    scale = (torch.rand(K, generator=g) * 0.5 + 0.1).cuda() if affine else None
    shift = torch.randn(K, generator=g).cuda() if affine else None
    got = []
    for kernel in (1, 0):
        codes = torch.full((B.dsq_act_packed_bytes(N, Ho, Wo, K, bits_next),), 0x5A, dtype=torch.uint8, device="cuda")
        sums = torch.full((N * Ho * Wo,), -3, dtype=torch.int32, device="cuda")
        B.dsq_conv2d_requant(_desc(geom, bits, next_flag | B.DSQ_CONV_KERNEL(kernel)), buf.act_packed, buf.pix_code_sum, la, 2.5,
                             buf.w_packed, buf.w_aux, scale, shift, True, 0.0, 40.0, bits_next, codes, sums)
        got.append((codes.cpu().numpy(), sums.cpu().numpy()))
    assert np.array_equal(got[1][0], got[0][0]) and np.array_equal(got[1][1], got[0][1])
    assert got[0][1].max() > 0


def test_what_the_rule_leaves_to_other_kernels():
    for geom, flags, chained in (((16, 64, 32, 32, 64, 3, 1, 1), 0, False),                          # 1024 tiles
                                 ((8, 256, 14, 14, 256, 3, 1, 1), 0, False),                         # 392 tiles of a deep 4-bit layer
                                 ((1, 64, 8, 8, 64, 3, 1, 1), B.DSQ_CONV_MANY_IN_FLIGHT, False),
                                 ((1, 64, 8, 8, 64, 3, 1, 1), 0, True),                              # whole pixel sums in one workgroup
                                 ((1, 576, 8, 8, 64, 3, 1, 1), B.DSQ_CONV_NEXT_SUMS_ZERO, True)):
        assert B.dsq_conv2d_plan(_desc(geom, 4, flags), chained=chained).startswith("patch kernel"), geom
