"""dsq_conv2d_wq (quantized weights, binary32 activations: the "b/32" rows of the
paper's Tables 3, 6 and 7) against the oracle's float64 convolution of the
activations with the weight levels.

Tolerance: the kernel sums K = R*S*C_in products of centred codes and activations,
exact on the bf16 matrix instruction (each activation in three parts), in binary32,
and combines them with the channel's step and offset in one rounding each (tiles that
cannot be split so: levels formed with one binary32 rounding, fp32 matrix
instruction).  So |gpu - ref| <= (K + 2) * 2^-24 * sum|a * w_hat|
(the classical bound of a length-K recursive sum); the tests demand that bound
and, as a sharper statistical check, a root-mean-square error below
4 * sqrt(K) * 2^-24 of the root-mean-square of that scale."""
import numpy as np
import pytest
import torch

import oracle
from paper_1908_05033_amd import binding as B
from paper_1908_05033_amd import inputs

pytestmark = pytest.mark.gpu


def run_wq(layer, x_nchw, w, lw, uw, bits, x_layout=B.DSQ_NHWC, out_layout=B.DSQ_NHWC, w_codes=None):
    L = layer
    d = B.make_desc(L.N, L.C_in, L.H, L.W, L.C_out, L.R, L.S, L.stride, L.pad, bits)
    wp = torch.empty(B.dsq_wgt_packed_bytes(L.C_out, L.C_in, L.R, L.S, 4), dtype=torch.uint8, device="cuda")
    aux = torch.empty(B.dsq_wgt_aux_bytes(L.C_out, L.R, L.S), dtype=torch.uint8, device="cuda")
    B.dsq_pack_weights_for(w.contiguous().cuda() if w_codes is None else None, torch.from_numpy(lw).cuda(),
                           torch.from_numpy(uw).cuda(), None if w_codes is None else torch.from_numpy(w_codes).cuda(),
                           L.C_out, L.C_in, L.R, L.S, bits, 4, wp, aux)
    xd = (x_nchw.permute(0, 2, 3, 1) if x_layout == B.DSQ_NHWC else x_nchw).contiguous().cuda()
    shape = (L.N, L.Ho, L.Wo, L.C_out) if out_layout == B.DSQ_NHWC else (L.N, L.C_out, L.Ho, L.Wo)
    out = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    B.dsq_conv2d_wq(d, xd, x_layout, wp, aux, out, out_layout)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    return o.transpose(0, 3, 1, 2) if out_layout == B.DSQ_NHWC else o


def check(got, ref, scale, K):
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    # (two roundings on the subnormal grid, of the output and of the reference)
    bound = (K + 2) * 2.0 ** -24 * scale.astype(np.float64) + 2.0 ** -149
    assert (err <= bound).all(), "worst error %.3e (largest bound %.3e)" % (err.max(), bound.max())
    rms = np.sqrt(np.mean(err ** 2))
    assert rms <= 4 * np.sqrt(K) * 2.0 ** -24 * np.sqrt(np.mean(scale.astype(np.float64) ** 2))


SMALL = [  # N, C_in, H, W, C_out, R, stride, pad
    (2, 64, 9, 7, 64, 3, 1, 1),
    (1, 24, 10, 11, 144, 1, 1, 0),
    (3, 144, 5, 6, 24, 1, 1, 0),
    (2, 96, 7, 9, 40, 3, 2, 1),
    (5, 70, 7, 7, 33, 3, 1, 1),
    (1, 3, 12, 12, 8, 3, 1, 1),
    (1, 64, 4, 150, 32, 3, 1, 2),
    (2, 130, 6, 5, 300, 1, 2, 0),
    (4, 512, 1, 1, 10, 1, 1, 0),
]


@pytest.mark.parametrize("layouts", [(B.DSQ_NHWC, B.DSQ_NHWC), (B.DSQ_NCHW, B.DSQ_NCHW), (B.DSQ_NHWC, B.DSQ_NCHW)])
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("geom", SMALL)
def test_small_geometries(geom, bits, layouts):
    N, Ci, H, W, Co, R, stride, pad = geom
    layer, inp = inputs.small_random_case(sum(geom) + bits, N, Ci, H, W, Co, R, stride, pad, 4, l_a=-1.0, u_a=1.0)
    x = inp["x"]                                           # real-valued activations, both signs
    code = oracle.quantize_weights(inp["w"].numpy(), inp["l_w"], inp["u_w"], bits)
    ref, scale = oracle.conv_weight_only(x.numpy(), code, inp["l_w"], inp["u_w"], bits, stride, pad)
    got = run_wq(layer, x, inp["w"], inp["l_w"], inp["u_w"], bits, *layouts)
    check(got, ref, scale, Ci * R * R)


def test_binary_weights_give_the_scaled_convolution_of_signs_exactly():
    """Integer-valued activations and (l, u) = (-alpha, +alpha) with alpha a power of two:
    every product and every partial sum is exact in binary32, so the output must be
    alpha * conv(x, sgn(w)) bit for bit."""
    import torch.nn.functional as F
    layer, inp = inputs.small_random_case(9, 2, 192, 9, 8, 80, 3, 1, 1, 1)
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.integers(-8, 9, (2, 192, 9, 8)).astype(np.float32))
    alpha = np.full(80, 0.25, np.float32)
    got = run_wq(layer, x, inp["w"], -alpha, alpha, 1)
    sgn = torch.where(inp["w"] >= 0, 1.0, -1.0).double()
    want = (F.conv2d(x.double(), sgn, padding=1) * 0.25).numpy()
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("bits,li", [(1, 0), (1, 5), (2, 8), (1, 3)])
def test_resnet18_layers_at_full_size(bits, li):
    """The 1/32 and 2/32 rows of Table 7 are ResNet-18: its layer shapes at batch 64,
    every output element."""
    layer, inp = inputs.make_config_layer(3, li, bits=4)
    L = layer
    x = inp["x"] - 0.8                                      # real-valued activations of both signs
    code = oracle.quantize_weights(inp["w"].numpy(), inp["l_w"], inp["u_w"], bits)
    ref, scale = oracle.conv_weight_only(x.numpy(), code, inp["l_w"], inp["u_w"], bits, L.stride, L.pad)
    got = run_wq(layer, x, inp["w"], inp["l_w"], inp["u_w"], bits)
    check(got, ref, scale, L.C_in * L.R * L.S)


def test_argument_errors():
    d = B.make_desc(1, 64, 4, 4, 64, 3, 3, 1, 1, 2)
    x = torch.zeros((1, 4, 4, 64), device="cuda")
    wp = torch.zeros(B.dsq_wgt_packed_bytes(64, 64, 3, 3, 4), dtype=torch.uint8, device="cuda")
    aux = torch.zeros(B.dsq_wgt_aux_bytes(64, 3, 3), dtype=torch.uint8, device="cuda")
    out = torch.zeros((1, 4, 4, 64), device="cuda")
    for args, status in (((d, None, 0, wp, aux, out, 0), 1), ((d, x, 0, wp, aux, None, 0), 1), ((d, x, 3, wp, aux, out, 0), 5),
                         ((d, x, 0, wp, aux, out, 2), 5)):
        with pytest.raises(B.DsqError) as e:
            B.dsq_conv2d_wq(*args)
        assert e.value.status == status
    d2 = B.make_desc(1, 64, 4, 4, 64, 3, 3, 1, 1, 2, B.DSQ_CONV_KERNEL(1))
    with pytest.raises(B.DsqError) as e:
        B.dsq_conv2d_wq(d2, x, 0, wp, aux, out, 0)
    assert e.value.status == 5
