"""The staged convolution kernel (k <= 3) at the geometries where its tiles,
its staged rows and its channel chunks can go wrong: grids below and above a
tile, several images in a tile, chunks of fewer than 8 channels, the four
output phases of stride 2 and the one tap per phase of k = s = 3, large
dilations, both kernel types; and values that the split cannot carry."""

import numpy as np
import pytest
import torch

from oracle import checks, conv
from paper_2601_13776_amd import orth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
REL = 1e-5   # fp32 sums over at most c k^2 = 1200 terms (measured: below 1e-6)

CASES = [  # (cin, cout, k, s, d, g), batch, H, W
    ((8, 64, 3, 1, 1, 1), 3, 5, 7), ((9, 65, 3, 1, 1, 1), 2, 16, 8), ((2, 3, 3, 1, 1, 1), 2, 6, 6),
    ((7, 130, 3, 1, 1, 1), 1, 33, 31), ((20, 12, 3, 1, 1, 2), 5, 3, 3), ((17, 5, 2, 1, 1, 1), 2, 9, 10),
    ((15, 66, 1, 1, 1, 1), 4, 13, 12), ((33, 40, 1, 1, 1, 1), 1, 1, 1), ((16, 24, 2, 1, 3, 2), 2, 12, 10),
    # stride 2: forward, and the transposed form's four output phases
    ((16, 64, 2, 2, 1, 1), 3, 8, 12), ((5, 21, 2, 2, 3, 1), 2, 10, 14), ((24, 70, 3, 2, 1, 1), 2, 18, 22),
    ((12, 20, 3, 2, 3, 2), 3, 14, 10), ((66, 9, 3, 2, 1, 1), 1, 2, 2),
    # k = s = 3: one tap per output phase
    ((10, 35, 3, 3, 1, 1), 2, 12, 9), ((6, 8, 3, 3, 2, 2), 2, 9, 15),
    # stride 3 forward: most staged positions per thread
    ((9, 20, 3, 3, 1, 1), 3, 27, 27),
    # large dilations: staged rows per grid row; more than two positions per thread
    ((8, 16, 3, 1, 6, 1), 2, 33, 33), ((8, 8, 3, 1, 11, 1), 1, 40, 24), ((6, 16, 3, 1, 1, 1), 2, 40, 100),
    # past the staged positions: the direct kernel
    ((3, 4, 3, 1, 1, 1), 1, 4, 500),
]


def rand(shape, seed):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("geom,b,h,w", CASES)
def test_parity(geom, b, h, w, dtype):
    cin, cout, k, s, d, g = geom
    kt = torch.from_numpy(rand((cout, cin // g, k, k), 1)).to(DEV)
    if dtype == "bf16":
        kt = kt.to(torch.bfloat16)
    k64 = kt.double().cpu().numpy()
    x = rand((b, cin, h, w), 2)
    y = orth.orth_conv_apply(kt, geom, torch.from_numpy(x).to(DEV))
    ref = conv.conv_circular(k64, x.astype(np.float64), s, d, g)
    assert checks.relative_difference(y.cpu().numpy().astype(np.float64), ref) <= REL
    yy = rand((b, cout, h // s, w // s), 3)
    z = orth.orth_conv_apply(kt, geom, torch.from_numpy(yy).to(DEV), transposed=True)
    ref = conv.conv_circular_adjoint(k64, yy.astype(np.float64), (h, w), s, d, g)
    assert checks.relative_difference(z.cpu().numpy().astype(np.float64), ref) <= REL


# an infinite or NaN input reaches exactly the outputs whose window holds it,
# an input near the fp32 limit keeps its value (it rounds to a bfloat16
# infinity), and the rest of the tile is ordinary
@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 3.399e38])
def test_extreme_inputs(bad, stride, transposed):
    geom, h = (12, 20, 3, stride, 1, 1), 12
    kern = np.abs(rand((20, 12, 3, 3), 4)) * 0.05 + 0.01
    kt = torch.from_numpy(kern.astype(np.float32)).to(DEV)
    x = rand((2, 20, h // stride, h // stride) if transposed else (2, 12, h, h), 5)
    x[1, 3, 2, 4] = 0.0
    run = lambda v: orth.orth_conv_apply(kt, geom, torch.from_numpy(v).to(DEV), transposed=transposed).cpu().numpy()
    base = run(x)
    hit = np.zeros_like(x)
    hit[1, 3, 2, 4] = 1.0
    hit = run(hit) != 0
    x[1, 3, 2, 4] = bad
    got = run(x)
    # (a wave with a non-finite result computes its block with fp32 products:
    # the others of the block differ by the rounding of at most 180-term sums)
    assert np.allclose(got[~hit], base[~hit], rtol=0, atol=1e-6 * np.abs(base).max() * 4)
    if np.isnan(bad):
        assert np.isnan(got[hit]).all()
    elif np.isinf(bad):
        assert np.isposinf(got[hit]).all()
    else:
        ref = np.zeros_like(x, dtype=np.float64)
        ref[1, 3, 2, 4] = np.float32(bad)
        k64 = kern.astype(np.float32).astype(np.float64)
        ref = conv.conv_circular_adjoint(k64, ref, (h, h), stride) if transposed else conv.conv_circular(k64, ref, stride)
        assert np.allclose(got[hit].astype(np.float64), ref[hit], rtol=1e-6)


# one infinite input at every geometry: the tiles that meet it are computed
# again with fp32 products, and everything outside its window is what it was
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("geom,b,h,w", CASES)
def test_nonfinite_geometries(geom, b, h, w, dtype):
    cin, cout, k, s, d, g = geom
    kt = torch.from_numpy(rand((cout, cin // g, k, k), 6)).to(DEV)
    if dtype == "bf16":
        kt = kt.to(torch.bfloat16)
    k64 = kt.double().cpu().numpy()
    for transposed in (False, True):
        x = rand((b, cout, h // s, w // s) if transposed else (b, cin, h, w), 7)
        at = tuple(v - 1 - (v > 2) for v in x.shape)   # in the last channels, off the corner
        apply64 = lambda kk, v: (conv.conv_circular_adjoint(kk, v, (h, w), s, d, g) if transposed else   # noqa: E731
                                 conv.conv_circular(kk, v, s, d, g))
        x[at] = 0.0
        ref = apply64(k64, x.astype(np.float64))
        one = np.zeros_like(x, dtype=np.float64)
        one[at] = 1.0
        hit = apply64(np.abs(k64), one) > 0
        x[at] = np.inf
        got = orth.orth_conv_apply(kt, geom, torch.from_numpy(x).to(DEV), transposed=transposed).cpu().numpy()
        assert not np.isfinite(got[hit]).any() and hit.any()
        if not hit.all():
            assert checks.relative_difference(got[~hit][None].astype(np.float64), ref[~hit][None]) <= REL


# inputs near the low end of fp32 keep its accuracy (their low pieces would
# not; the tiles are computed with fp32 products)
@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("exp", [-104, -120])
def test_small_inputs(exp, transposed):
    geom = (16, 24, 3, 2, 1, 1)
    kern = rand((24, 16, 3, 3), 8)
    x = rand((2, 24, 6, 6) if transposed else (2, 16, 12, 12), 9) * np.float32(2.0 ** exp)
    got = orth.orth_conv_apply(torch.from_numpy(kern).to(DEV), geom, torch.from_numpy(x).to(DEV),
                               transposed=transposed).cpu().numpy().astype(np.float64)
    k64, x64 = kern.astype(np.float64), x.astype(np.float64)
    ref = conv.conv_circular_adjoint(k64, x64, (12, 12), 2) if transposed else conv.conv_circular(k64, x64, 2)
    assert checks.relative_difference(got * 2.0 ** -exp, ref * 2.0 ** -exp) <= 1e-6   # (fp32 sums of 144 terms)
