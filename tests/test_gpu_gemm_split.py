"""fp32 products on 16-bit matrix cores: the sizes where the tiles, the
K-steps and the choice of tile edge can go wrong, inputs whose parts differ
by many powers of two (every part keeps fp32's relative accuracy), the
values that the split cannot carry (infinities, overflow), and the scaling
of gradients."""

import numpy as np
import pytest
import torch

from oracle import aoc, aoc_grad, bjorck, bjorck_grad, checks, expo, spectral
from paper_2601_13776_amd import orth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-5   # fp32 products against the float64 oracle (measured: below 1e-6)


def _rand(seed, *shape):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


def _run(mats, iters, **kw):
    ins = [torch.from_numpy(m).to(DEV) for m in mats]
    outs = [torch.empty_like(t) for t in ins]
    orth.orth_orthogonalize_batched(ins, outs, iters, **kw)
    return [t.cpu().numpy().astype(np.float64) for t in outs]


# 64-tiles: K of whole steps only, with a remainder, below one step; rows at
# the edges of tiles
@pytest.mark.parametrize("shape", [(129, 3), (129, 31), (160, 65), (64, 200), (191, 96), (257, 127), (128, 65)])
def test_small_lists(shape):
    m = _rand(1, *shape)
    got = _run([m], 8)[0]
    assert checks.relative_difference(got, bjorck.bjorck(m.astype(np.float64), 8)) <= TOL


# enough 128-tiles for every compute unit: the 128-tile kernel, on shapes
# that fill and that overhang its tiles
@pytest.mark.parametrize("shape,n", [((512, 512), 16), ((500, 449), 16), ((130, 1030), 18), ((321, 640), 18)])
@pytest.mark.parametrize("prescale", ["frobenius", "none"])
def test_big_tile_lists(shape, n, prescale):
    rng = np.random.default_rng(2)
    mats = [(rng.standard_normal(shape) * (0.02 if prescale == "none" else 3.0)).astype(np.float32) for _ in range(n)]
    got = _run(mats, 6, prescale=prescale)
    for i in (0, n - 1):
        ref = bjorck.bjorck(mats[i].astype(np.float64), 6, prescale=prescale)
        assert checks.relative_difference(got[i], ref) <= TOL


# a strided view whose row offsets within a tile exceed 32 bits (in bytes):
# rows and k-major; each row of the tile is its own
@pytest.mark.parametrize("rows,cols,ld", [(64, 100, 17_100_000), (72, 40, 36_000_000)])
def test_gram_of_long_strides(rows, cols, ld):
    m = _rand(12, rows, cols)
    buf = torch.zeros(rows, ld, device=DEV)
    view = buf[:, :cols]
    view.copy_(torch.from_numpy(m))
    got = float(orth.orth_check_norm_gram([view])[0])
    ref = checks.gram_deviation(m.astype(np.float64))
    assert abs(got - ref) <= TOL * max(1.0, ref)


# bfloat16 operands (their own leading piece): rows and k-major, whole steps
# and remainders, tiles that end on a multiple of four rows and that do not,
# views that are only 2-byte aligned
@pytest.mark.parametrize("shape", [(96, 64), (64, 96), (100, 68), (72, 300), (257, 33), (130, 131), (320, 130)])
@pytest.mark.parametrize("offset", [0, 1])
def test_gram_of_bf16(shape, offset):
    buf = torch.from_numpy(_rand(17, shape[0], shape[1] + 3)).to(DEV).to(torch.bfloat16)
    view = buf[:, offset:offset + shape[1]]
    got = float(orth.orth_check_norm_gram([view])[0])
    ref = checks.gram_deviation(view.double().cpu().numpy())
    assert abs(got - ref) <= TOL * max(1.0, ref)


# an infinity in bfloat16 matrices (their blocks run on fp32 products), also
# where two of them lie in each 4 bytes of a k-major operand
@pytest.mark.parametrize("shape", [(40, 2), (100, 68), (64, 96)])
def test_gram_of_bf16_infinite(shape):
    m = torch.from_numpy(np.abs(_rand(18, *shape)) + 0.1).to(DEV).to(torch.bfloat16)
    m[3, 1] = float("inf")
    assert float(orth.orth_check_norm_gram([m])[0]) == float("inf")


# light rows keep their own relative accuracy beside rows 2^10 times larger
def test_row_scales():
    m = _rand(3, 192, 128)
    m[::7] *= 1024.0
    got = _run([m], 5)[0]
    ref = bjorck.bjorck(m.astype(np.float64), 5)
    light = np.arange(192) % 7 != 0
    assert checks.relative_difference(got[light], ref[light]) <= TOL


# and at any ratio, before and at convergence (a light column grows by at
# most 3/2 a step, so 2^-30 needs more than 51 of them)
@pytest.mark.parametrize("prescale", ["frobenius", "spectral"])
@pytest.mark.parametrize("exp", [-20, -24, -30])
def test_light_rows_and_columns(exp, prescale):
    def run(m, iters):
        u = _rand(14, min(m.shape))
        kw = dict(u=torch.from_numpy(u.copy()).to(DEV), power_iters=4) if prescale == "spectral" else {}
        got = _run([m], iters, prescale=prescale, **kw)[0]
        m64 = m.astype(np.float64)
        return got, (spectral.bjorck_spectral(m64, u.astype(np.float64), iters, 4)[0] if kw else
                     bjorck.bjorck(m64, iters))
    for shape in [(192, 128), (513, 256), (130, 300)]:
        m = _rand(13, *shape)
        m[::7] *= np.float32(2.0 ** exp)
        got, ref = run(m, 12)
        light = np.arange(shape[0]) % 7 == 0
        for rows in (light, ~light):
            assert checks.relative_difference(got[rows], ref[rows]) <= TOL, (shape, "rows")
        m = _rand(15, *shape)
        m[:, ::7] *= np.float32(2.0 ** exp)
        light = np.arange(shape[1]) % 7 == 0
        for iters in (12, 70):
            got, ref = run(m, iters)
            for cols in (light, ~light):
                assert checks.relative_difference(got[:, cols], ref[:, cols]) <= TOL, (shape, "columns", iters)


# gradients of two uncoupled blocks that differ by 2^exp (the cached vector
# lies in the first one, whose leading singular value sets sigma): each
# block's gradient keeps its own relative accuracy
@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("exp", [-20, -30])
def test_light_gradient_block(exp, saved):
    m, g = np.zeros((192, 128), np.float32), np.zeros((192, 128), np.float32)
    u = np.zeros(128, np.float32)
    a, b = _rand(40, 96), _rand(41, 64)
    m[:96, :64] = _rand(42, 96, 64) + 60.0 * np.outer(a / np.linalg.norm(a), b / np.linalg.norm(b))
    m[96:, 64:] = _rand(43, 96, 64)
    u[:64] = _rand(44, 64)
    g[:96, :64] = _rand(45, 96, 64)
    g[96:, 64:] = _rand(46, 96, 64) * np.float32(2.0 ** exp)
    w, go, ut = (torch.from_numpy(v).to(DEV) for v in (m, g, u.copy()))
    out = torch.empty_like(w)
    kw = dict(prescale="spectral", power_iters=2)
    ws = orth.orth_orthogonalize_save_batched([w], [torch.empty_like(w)], 6, u=ut, **kw) if saved else None
    orth.orth_orthogonalize_vjp_batched([w], [go], [out], 6, u=None if saved else ut, workspace=ws, saved=saved, **kw)
    got = out.cpu().numpy().astype(np.float64)
    m64, g64 = m.astype(np.float64), g.astype(np.float64)
    ref = spectral.bjorck_spectral_vjp(m64, u.astype(np.float64), g64, 6, 2)
    for rows, cols in ((slice(0, 96), slice(0, 64)), (slice(96, 192), slice(64, 128))):
        assert checks.relative_difference(got[rows, cols], ref[rows, cols]) <= TOL


# an infinity comes out as fp32 arithmetic has it, and a value that rounds to
# a bfloat16 infinity keeps its fp32 result, on row-major and odd-sized
# products
@pytest.mark.parametrize("c,og", [(64, 64), (37, 29)])
def test_nonfinite_products(c, og):
    rko = _rand(4, 1, og, c)
    rko[0, 3, 5] = np.inf
    rko[0, 7] = 0.0
    rko[0, 7, 2] = np.float32(3.399e38)
    proj = (_rand(5, 1, 2, c, c // 2) / np.sqrt(2.0 * c)).astype(np.float32)
    R, P = torch.from_numpy(rko).to(DEV), torch.from_numpy(proj).to(DEV)
    K = torch.empty(og, c, 2, 2, device=DEV)
    orth.orth_build_conv_kernels_batched([dict(geom=(c, og, 2, 1, 1, 1), rko=R, proj=P, kernel=K)])
    got = K.cpu().numpy()

    def compose(t, p):
        y = t @ p[0]
        h = [y, t - y]
        return np.stack([np.stack([h[b] @ p[1] for b in range(2)]),
                         np.stack([h[b] - h[b] @ p[1] for b in range(2)])]).transpose(2, 3, 0, 1)
    with np.errstate(all="ignore"):
        ref = compose(rko[0], [v @ v.T for v in proj[0]])
        v64 = proj[0].astype(np.float64)
        ref64 = compose(np.nan_to_num(rko[0].astype(np.float64), posinf=0.0), [v @ v.T for v in v64])
    assert np.array_equal(np.isnan(got[3]), np.isnan(ref[3])) and not np.isfinite(got[3]).any()
    for rows in ([o for o in range(og) if o not in (3, 7)], [7]):
        assert np.isfinite(got[rows]).all()
        scale = np.abs(ref64[rows]).max()
        assert checks.relative_difference(got[rows] / scale, ref64[rows] / scale) <= TOL


# compositions and their VJP with enough 128-tiles for every compute unit:
# k-major products with ragged M and N (388) and ones that are no multiple of
# four (387), row-major ones with a remainder of K (194, 193), fp32 and
# bfloat16 operands, whole and per 128-block; a layer of non-finite values
# (on fp32 products) leaves the others alone
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c", [388, 387])
def test_big_tile_compositions(c, dtype):
    n, geom, tol = 16, (c, c, 3, 1, 1, 1), TOL if dtype == "f32" else 4e-3   # one bfloat16 rounding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    dev = lambda a: torch.from_numpy(a).to(DEV).to(dt).contiguous()   # noqa: E731
    rko = [_rand(60 + i, 1, c, c) for i in range(n)]
    proj = [(_rand(80 + i, 1, 4, c, c // 2) / np.sqrt(c)).astype(np.float32) for i in range(n)]
    dk = [_rand(100 + i, c, c, 3, 3) for i in range(n)]
    bad = 5
    rko[bad][0, 7, 3] = np.inf
    dk[bad][9, 4, 1, 1] = np.nan
    layers = [dict(geom=geom, rko=dev(r), proj=dev(p), kernel=torch.empty(c, c, 3, 3, dtype=dt, device=DEV),
                   grad_kernel=dev(g), grad_rko=torch.empty(1, c, c, dtype=dt, device=DEV),
                   grad_proj=torch.empty(1, 4, c, c // 2, dtype=dt, device=DEV))
              for r, p, g in zip(rko, proj, dk)]
    orth.orth_build_conv_kernels_batched(layers)
    orth.orth_build_conv_kernels_vjp_batched(layers)
    f64 = lambda t: t.double().cpu().numpy()   # noqa: E731
    for i in (0, n - 1):
        L = layers[i]
        r64, p64, g64 = f64(L["rko"]), f64(L["proj"]), f64(L["grad_kernel"])
        got = f64(L["kernel"])
        ref = aoc.aoc_kernel(r64, p64, *geom)
        pairs = [(got[:, :, a, b], ref[:, :, a, b]) for a in range(3) for b in range(3)]
        dr, dp = aoc_grad.aoc_kernel_vjp(r64, p64, *geom, g64)
        pairs += [(f64(L["grad_rko"])[0], dr[0])]
        pairs += [(f64(L["grad_proj"])[0, t], dp[0, t]) for t in range(4)]
        for a, b in pairs:
            assert checks.tile_relative_differences(a, b, 128).max() <= tol
    for i, L in enumerate(layers):
        fin = [bool(torch.isfinite(L[k]).all()) for k in ("kernel", "grad_rko", "grad_proj")]
        assert fin == [i != bad] * 3, (i, fin)
    rows = torch.isfinite(layers[bad]["kernel"].float()).flatten(1).all(1)
    assert rows.sum() == c - 1 and not rows[7]


# values near the low end of fp32 keep its accuracy without pre-scaling: E is
# the identity to fp32, so a step multiplies them by 3/2
def test_small_values():
    m = _rand(16, 192, 130) * np.float32(2.0 ** -120)
    got = _run([m], 3, prescale="none")[0]
    assert checks.relative_difference(got * 2.0 ** 120, m.astype(np.float64) * (2.0 ** 120 * 3.375)) <= 1e-6


# gradients of any power-of-two scale give the same result times that scale,
# bit for bit (the products scale them themselves)
@pytest.mark.parametrize("exp", [-90, -23, 17, 60])
def test_gradient_scale(exp):
    mats = [_rand(6, 150, 97), _rand(7, 96, 256)]
    ws = [torch.from_numpy(m).to(DEV) for m in mats]
    grads = [torch.from_numpy(_rand(8 + i, *m.shape)).to(DEV) for i, m in enumerate(mats)]

    def vjp(gs):
        out = [torch.empty_like(w) for w in ws]
        orth.orth_orthogonalize_vjp_batched(ws, gs, out, 5)
        return out
    one = vjp(grads)
    other = vjp([g * 2.0 ** exp for g in grads])
    for a, b, m, g in zip(one, other, mats, grads):
        assert torch.equal(a * 2.0 ** exp, b)
        ref = bjorck_grad.bjorck_vjp(m.astype(np.float64), g.cpu().numpy().astype(np.float64), 5)
        assert checks.relative_difference(a.cpu().numpy().astype(np.float64), ref) <= TOL


# a NaN or an infinity in one gradient leaves the other matrices alone
def test_gradient_nonfinite():
    mats = [_rand(9, 130, 70), _rand(10, 130, 70)]
    ws = [torch.from_numpy(m).to(DEV) for m in mats]
    grads = [torch.from_numpy(_rand(11 + i, 130, 70)).to(DEV) for i in range(2)]
    ref = [torch.empty_like(w) for w in ws]
    orth.orth_orthogonalize_vjp_batched(ws, grads, ref, 4)
    for bad in (float("nan"), float("inf")):
        g = [grads[0].clone(), grads[1]]
        g[0][5, 6] = bad
        out = [torch.empty_like(w) for w in ws]
        orth.orth_orthogonalize_vjp_batched(ws, g, out, 4)
        assert not torch.isfinite(out[0]).all()
        assert torch.equal(out[1], ref[1])


# iterates and powers that grow: the estimate of sigma misses a heavy block
# (the cached vector has no part in it), so the iterates of a few steps and
# the powers leave the range that a good estimate gives them
def _heavy(c, heavy):
    m = _rand(20, c, c)
    m[:, -heavy:] = 0.0
    m[-heavy:, :] = 0.0
    m[-heavy:, -heavy:] = 1000.0 * _rand(21, heavy, heavy)
    u = _rand(22, c)
    u[-heavy:] = 0.0
    return m, u


@pytest.mark.parametrize("c,heavy,iters", [(200, 6, 1), (300, 10, 2), (129, 3, 2), (300, 10, 3)])
def test_diverging_spectral(c, heavy, iters):
    m, u = _heavy(c, heavy)
    got = _run([m], iters, prescale="spectral", u=torch.from_numpy(u.copy()).to(DEV))[0]
    ref, _, _ = spectral.bjorck_spectral(m.astype(np.float64), u.astype(np.float64), iters, 1)
    assert np.abs(ref).max() > 200
    assert checks.relative_difference(got, ref) <= TOL


@pytest.mark.parametrize("c,heavy,terms", [(512, 2, 8), (450, 2, 9), (2000, 2, 12)])
def test_exp_map_poor_sigma(c, heavy, terms):
    m, u = _heavy(c, heavy)
    w = torch.from_numpy(m).to(DEV)
    out = torch.empty_like(w)
    orth.orth_exp_map_batched([w], [out], terms, torch.from_numpy(u.copy()).to(DEV), 1)
    ref, _ = expo.exp_map(m.astype(np.float64), terms, u.astype(np.float64))
    assert np.abs(ref).max() > 65504
    assert checks.relative_difference(out.cpu().numpy().astype(np.float64), ref) <= TOL


# light channels of the exponentials: rows and columns 2^-30 times the
# others' keep their own relative accuracy off the diagonal
@pytest.mark.parametrize("c", [96, 200])
def test_exp_light_channels(c):
    light = np.arange(c) % 5 == 0
    f = np.where(light, np.float32(2.0 ** -30), np.float32(1.0))
    m, u = _rand(50, c, c) * f[:, None] * f, _rand(51, c) * f
    out = torch.empty(c, c, device=DEV)
    orth.orth_exp_map_batched([torch.from_numpy(m).to(DEV)], [out], 8, torch.from_numpy(u.copy()).to(DEV), 2)
    ref, _ = expo.exp_map(m.astype(np.float64), 8, u.astype(np.float64), 2)
    got = out.cpu().numpy().astype(np.float64)
    assert checks.relative_difference(got[~light][:, light], ref[~light][:, light]) <= TOL
    assert checks.relative_difference(got[light][:, ~light], ref[light][:, ~light]) <= TOL
    kern = _rand(52, c, c, 3, 3) * (f[:, None] * f)[:, :, None, None]
    co = torch.empty(c, c, 7, 7, device=DEV)
    orth.orth_conv_exp_batched([dict(kernel=torch.from_numpy(kern).to(DEV), out=co, terms=3, scale=0.02)])
    ref = expo.conv_exp(kern.astype(np.float64), 3, float(np.float32(0.02)))
    got = co.cpu().numpy().astype(np.float64)
    assert checks.relative_difference(got[~light][:, light], ref[~light][:, light]) <= TOL
    assert checks.relative_difference(got[light][:, ~light], ref[light][:, ~light]) <= TOL


# conv exponentials: channel counts at the edges of the padded rows and
# tiles (the last one fills every compute unit with 128-tiles), series of 2
# and 3 terms, kernels of any size
@pytest.mark.parametrize("c,k,terms,scale", [(31, 3, 3, 0.05), (33, 5, 4, 0.1), (65, 3, 2, 0.02), (96, 1, 5, 0.05),
                                             (512, 3, 3, 0.004), (40, 3, 4, 40.0), (16, 5, 3, 1e8),
                                             (24, 3, 4, 1e-9)])
def test_conv_exp_pieces(c, k, terms, scale):
    kern = _rand(30, c, c, k, k)
    S = terms * (k - 1) + 1
    out = torch.full((c, c, S, S), float("nan"), device=DEV)
    orth.orth_conv_exp_batched([dict(kernel=torch.from_numpy(kern).to(DEV), out=out, terms=terms, scale=scale)])
    got = out.cpu().numpy().astype(np.float64)
    ref = expo.conv_exp(kern.astype(np.float64), terms, float(np.float32(scale)))
    assert checks.relative_difference(got, ref) <= TOL
    if scale < 1e-6:   # the kernel itself, beside the identity
        eye = np.zeros_like(ref)
        eye[np.arange(c), np.arange(c), S // 2, S // 2] = 1.0
        off = ~(eye > 0)
        assert checks.relative_difference(got[off][None], ref[off][None]) <= TOL


# Blocks that the split cannot give run on fp32 MFMA after it: 16 / 6 of its
# time at the same efficiency, 3.7 with the first pass.  Calls with one
# non-finite value among their operands stay within 8 times (an element load
# per lane and step took 10 to 26 times).
def _time(f):
    for _ in range(3):
        f()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ms = []
    for _ in range(5):
        e[0].record()
        for _ in range(4):
            f()
        e[1].record()
        torch.cuda.synchronize()
        ms.append(e[0].elapsed_time(e[1]))
    return sorted(ms)[2]


@pytest.mark.parametrize("what", ["conv_exp", "conv", "conv_transposed"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_cost_of_blocks_computed_again(what, bad):
    if what == "conv_exp":
        c, kern = 256, torch.from_numpy(_rand(70, 256, 256, 3, 3) / 48).to(DEV)
        layer = dict(kernel=kern, out=torch.empty(c, c, 13, 13, device=DEV), terms=6, scale=0.25)
        hit, run = kern[5, 7, 1], lambda: orth.orth_conv_exp_batched([layer])   # noqa: E731
    else:
        geom, tr = (128, 256, 3, 2, 1, 1), what == "conv_transposed"
        kern = torch.from_numpy(_rand(71, 256, 128, 3, 3) / 34).to(DEV)
        x = torch.from_numpy(_rand(72, 64, *((256, 16, 16) if tr else (128, 32, 32)))).to(DEV)
        hit, run = x[:, 3, 2], lambda: orth.orth_conv_apply(kern, geom, x, transposed=tr)   # noqa: E731
    plain = _time(run)
    hit[..., 1] = bad
    assert _time(run) <= 8 * plain
