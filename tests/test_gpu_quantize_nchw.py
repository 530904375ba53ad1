"""dsq_quantize_act on the shapes at the edges of its NCHW kernel (64 pixels of a plane, 64 packed
words of a pixel per pass, 4 or 16 waves) and of the kernel for few deep pixels: codes and code
sums against the oracle, with values on and beside the thresholds, infinities and NaN."""
import numpy as np
import pytest
import torch

import oracle
from helpers import unpack_act
from paper_1908_05033_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("layout,geom", [
    (B.DSQ_NCHW, (3, 5, 7, 9)), (B.DSQ_NCHW, (2, 128, 8, 8)), (B.DSQ_NCHW, (2, 130, 13, 5)), (B.DSQ_NCHW, (1, 1100, 3, 3)),
    (B.DSQ_NCHW, (70, 20, 64, 65)), (B.DSQ_NCHW, (5, 260, 1, 1)), (B.DSQ_NCHW, (2, 2050, 1, 3)),
    (B.DSQ_NCHW, (4200, 520, 3, 5)), (B.DSQ_NCHW, (4100, 130, 2, 2)),
    (B.DSQ_NHWC, (3, 8192, 1, 1)), (B.DSQ_NHWC, (2, 16388, 1, 1)), (B.DSQ_NHWC, (1, 70000, 1, 2)), (B.DSQ_NCHW, (3, 25088, 1, 1)),
])
def test_codes_and_sums(layout, geom, bits):
    N, C, H, W = geom
    l, u = -0.9, 2.1
    rng = np.random.default_rng(sum(geom) + bits)
    x = rng.normal(0.5, 1.2, (N, C, H, W)).astype(np.float32)
    flat = x.reshape(-1)
    delta = (np.float32(u) - np.float32(l)) / np.float32((1 << bits) - 1)
    edges = (np.float32(l) + (np.arange(1 << bits) + 0.5).astype(np.float32) * delta).astype(np.float32)
    special = np.concatenate([edges, np.nextafter(edges, np.float32(np.inf)), np.nextafter(edges, np.float32(-np.inf)),
                              np.array([np.inf, -np.inf, np.nan, l, u, 0.0, -0.0], np.float32)])
    at = rng.choice(flat.size, min(flat.size, special.size), replace=False)
    flat[at] = special[:at.size]
    want = oracle.quantize(x, l, u, bits)                        # [N, C, H, W]
    xd = torch.from_numpy(x if layout == B.DSQ_NCHW else np.ascontiguousarray(x.transpose(0, 2, 3, 1))).cuda()
    codes = torch.full((B.dsq_act_packed_bytes(N, H, W, C, bits),), 255, dtype=torch.uint8, device="cuda")
    sums = torch.full((N * H * W,), -7, dtype=torch.int32, device="cuda")
    B.dsq_quantize_act(xd, layout, N, C, H, W, l, u, bits, codes, sums)
    torch.cuda.synchronize()
    got = unpack_act(codes.cpu().numpy(), N, H, W, C, bits)
    want = want.transpose(0, 2, 3, 1)
    assert np.array_equal(got[..., :C], want)
    assert not got[..., C:].any()
    assert np.array_equal(sums.cpu().numpy(), want.reshape(N * H * W, C).astype(np.int64).sum(1))
