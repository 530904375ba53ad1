"""The LDS-patch kernel's plan against a walk over all of its tiles (CPU only): the patch must
hold the input rows of every tile, and little more."""
import random
import re

import pytest

from paper_1908_05033_amd import binding as B


def _rows_of_every_tile(N, H, Ho, stride, pad, R, TW, BP):
    rows, NHo, Hp = 0, N * Ho, H + 2 * pad
    for t in range(0, NHo * TW, BP):
        g0, g1 = t // TW, min((t + BP - 1) // TW, NHo - 1)
        first = g0 // Ho * Hp + g0 % Ho * stride
        last = g1 // Ho * Hp + g1 % Ho * stride
        rows = max(rows, last - first + R)
    return rows


@pytest.mark.parametrize("seed", range(6))
def test_patch_holds_the_rows_of_every_tile(seed):
    rng = random.Random(seed)
    planned = 0
    while planned < 60:
        R, stride = rng.choice([1, 3]), rng.choice([1, 2])
        pad, N = rng.randint(0, R - 1), rng.choice([1, 2, 3, 5, 17, 40])
        H, W = rng.choice([1, 2, 7, 14, 27, 53, 56, 101]), rng.choice([1, 3, 7, 14, 28, 53, 56, 113])
        if min(H, W) + 2 * pad < R:
            continue
        Ho = (H + 2 * pad - R) // stride + 1
        d = B.make_desc(N, rng.choice([16, 64, 200]), H, W, rng.choice([24, 64, 256]), R, R, stride, pad,
                        rng.choice([2, 4]), rng.choice([2, 3, 4, 5, 6]))
        try:
            text = B.dsq_conv2d_plan(d)
        except B.DsqError:
            continue                # the forced tile does not take this layer
        planned += 1
        BP = int(re.search(r"tile (\d+)x", text).group(1))
        TW = int(re.search(r"strip width (\d+)", text).group(1))
        PR = int(re.search(r"patch (\d+)x", text).group(1))
        need = _rows_of_every_tile(N, H, Ho, stride, pad, R, TW, BP)
        assert need <= PR <= need + 2, text


@pytest.mark.parametrize("seed", range(4))
def test_patch_is_no_higher_than_its_tiles_need(seed):
    """Exactly the rows of the worst tile: a row more costs LDS and fetch units, and the largest
    patches are then not taken.  (1x1, stride 2, odd height: one row more at most.)"""
    rng = random.Random(100 + seed)
    planned = 0
    while planned < 150:
        R, stride = rng.choice([1, 3, 3]), rng.choice([1, 2])
        pad, N = rng.randint(0, R - 1), rng.choice([1, 2, 3, 7, 16, 40])
        H, W = rng.randint(1, 120), rng.choice([rng.randint(1, 120), 32, 64, 96])
        if min(H, W) + 2 * pad < R:
            continue
        Ho = (H + 2 * pad - R) // stride + 1
        d = B.make_desc(N, rng.choice([16, 200]), H, W, rng.choice([24, 256]), R, R, stride, pad, rng.choice([2, 4]),
                        rng.choice([2, 3, 4, 5, 6]))
        try:
            text = B.dsq_conv2d_plan(d)
        except B.DsqError:
            continue
        planned += 1
        BP, TW, PR = (int(re.search(p, text).group(1)) for p in (r"tile (\d+)x", r"strip width (\d+)", r"patch (\d+)x"))
        need = _rows_of_every_tile(N, H, Ho, stride, pad, R, TW, BP)
        assert need <= PR <= need + (R == 1 and stride == 2 and H % 2), text


@pytest.mark.parametrize("geom,flags,rows", [((17, 200, 13, 125, 64, 3, 3, 1, 2, 2), 6, 7), ((64, 64, 3, 125, 256, 3, 3, 1, 2, 2), 6, 7),
                                             ((3, 64, 101, 224, 256, 3, 3, 2, 1, 4), 2, 9)])
def test_patch_rows_of_some_layers(geom, flags, rows):
    text = B.dsq_conv2d_plan(B.make_desc(*geom, B.DSQ_CONV_KERNEL(flags)))
    assert int(re.search(r"patch (\d+)x", text).group(1)) == rows, text


@pytest.mark.parametrize("geom,flags,l_a", [((300, 512, 2, 3, 64, 3, 3, 2, 2, 3), B.DSQ_CONV_ACT_DENSE3, -1.0),
                                            ((300, 512, 2, 224, 128, 3, 3, 2, 1, 3), B.DSQ_CONV_ACT_DENSE3, -1.0),
                                            ((300, 512, 1, 3, 300, 3, 3, 2, 2, 2), B.DSQ_CONV_KERNEL(6), -1.0)])
def test_largest_patches_are_taken_for_any_l_a(geom, flags, l_a):
    """The tables of a layer with l_a != 0 do not count against the patch."""
    d = B.make_desc(*geom, flags)
    assert B.dsq_conv2d_plan(d).startswith("patch kernel")
    assert B.dsq_conv2d_plan(d, l_a=l_a).startswith("patch kernel")
    assert int(re.search(r"(\d+) LDS bytes", B.dsq_conv2d_plan(d, l_a=l_a)).group(1)) <= 160 * 1024


@pytest.mark.parametrize("l_a", [0.0, -1.0])
def test_patches_past_the_limit_stay_refused(l_a):
    d = B.make_desc(17, 200, 14, 14, 24, 3, 3, 2, 2, 3, B.DSQ_CONV_ACT_DENSE3 | B.DSQ_CONV_KERNEL(5))
    with pytest.raises(B.DsqError) as e:
        B.dsq_conv2d_plan(d, l_a=l_a)
    assert e.value.status == 5
