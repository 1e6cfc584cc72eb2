"""Single layers at the sizes where the layer kernel's tiling and its split
fp32 operands can go wrong: list lengths around whole tiles, every channel
count, both strides, values far from 1, per-channel scales far apart, and
values that are not finite."""
import numpy as np
import pytest
import torch

import oracle
import streams as S
from gpu_util import note

pytestmark = pytest.mark.gpu


def _layer(cin, cout, stride, dtype, w, H=37, W=41, relu=False):
    from paper_2512_08557_amd import Engine
    return Engine(H, W, cin, [(cin, cout, stride, relu)], [w], dtype=dtype, max_pillars=H * W)


def _bf16(x):
    return S.bf16_bits_to_f32(S.round_to_bf16_bits(x)).reshape(x.shape)


def _window(rng, n, cin, H, W, scale, dtype):
    idx = np.sort(rng.choice(H * W, n, replace=False)).astype(np.int32)
    f = (rng.standard_normal((n, cin)) * scale).astype(np.float32)
    return idx, _bf16(f) if dtype == "bf16" else f


def _step(eng, win, dtype, sorted):
    idx, f = win
    t = torch.from_numpy(f)
    eng.step(torch.from_numpy(idx).cuda(), (t.bfloat16() if dtype == "bf16" else t).cuda(), sorted=sorted)


def _canvas(win, cin, H, W):
    x = np.zeros((H * W, cin))
    x[win[0]] = win[1]
    return x.reshape(H, W, cin)


def _conv(x, w, stride):
    return oracle.forward(x, [w], [(w.shape[1], w.shape[0], stride, False)])[0]


def _check(eng, wins, w, cin, stride, dtype, H, W, where):
    """|gpu - exact| per output, after the windows in turn.  Each stride adds a
    sum of K = 9*cin products to every touched cell.  fp32: a product of two
    split values is off by at most 3 * 2^-23 of itself, and summing takes at
    most one rounding per matrix instruction's 32 products, channel unit and
    wavefront (counted as 3 per unit, plus 16), 2^-24 each of the sum of
    magnitudes.  bf16 products are exact, and the output is rounded to bf16."""
    units = 9 * max(1, cin // 32)
    eps = (0 if dtype == "bf16" else 3 * 2.0 ** -23) + (3 * units + 16) * 2.0 ** -24
    xs = [_canvas(x, cin, H, W) for x in wins]
    ref = _conv(xs[-1], w, stride)
    mag = sum(_conv(np.abs(a) + np.abs(b), np.abs(w), stride) for a, b in zip([0 * xs[0]] + xs[:-1], xs))
    out = eng.read(1)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    tol = eps * mag + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    bad = np.abs(got - ref) > tol
    assert not bad.any(), f"{where}: {bad.sum()} outputs off, worst {np.abs(got - ref)[bad].max()}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("cin,cout", [(16, 8), (16, 64), (32, 16), (32, 256), (64, 32), (64, 64), (128, 8), (128, 128),
                                      (256, 64), (256, 256)])
def test_layer_shapes(cin, cout, stride, dtype):
    H, W = 37, 41
    rng = np.random.default_rng(cin * 1000 + cout + stride)
    w = (rng.standard_normal((cout, cin, 3, 3)) * (2.0 / (9 * cin)) ** 0.5).astype(np.float32)
    if dtype == "bf16":
        w = _bf16(w)
    eng = _layer(cin, cout, stride, dtype, w, H, W)
    wins = [_window(rng, n, cin, H, W, 1.0, dtype) for n in (1, 300, H * W, 40)]
    for k, win in enumerate(wins):
        note(f"[gpu-test] layer {cin}->{cout} s{stride} {dtype} window {k}")
        _step(eng, win, dtype, sorted=k % 2 == 0)
    _check(eng, wins, w, cin, stride, dtype, H, W, f"{cin}->{cout} s{stride} {dtype}")


@pytest.mark.parametrize("cells", [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 511])
def test_list_lengths_around_tiles(cells):
    """A stride-2 layer whose input cells are isolated and even: one output
    cell each, so the change list holds exactly `cells` entries."""
    H, W, c = 64, 64, 64
    rng = np.random.default_rng(cells)
    w = (rng.standard_normal((64, c, 3, 3)) * 0.06).astype(np.float32)
    eng = _layer(c, 64, 2, "f32", w, H, W)
    pos = rng.choice(32 * 32, cells, replace=False)
    idx = np.sort((pos // 32) * 2 * W + (pos % 32) * 2).astype(np.int32)
    win = (idx, rng.standard_normal((cells, c)).astype(np.float32))
    note(f"[gpu-test] list of {cells}")
    _step(eng, win, "f32", True)
    assert len(eng.changed(1)) == cells
    _check(eng, [win], w, c, 2, "f32", H, W, f"{cells} cells")


@pytest.mark.parametrize("cin", [16, 64, 256])
@pytest.mark.parametrize("fscale,wscale", [(1e-30, 1.0), (1e30, 1e-25), (1e-3, 1e-30), (3.0, 1e20)])
def test_magnitudes(cin, fscale, wscale):
    H, W = 37, 41
    rng = np.random.default_rng(cin)
    w = (rng.standard_normal((64, cin, 3, 3)) * wscale).astype(np.float32)
    w *= np.exp2(rng.integers(-6, 7, (64, 1, 1, 1))).astype(np.float32)      # output channels apart
    eng = _layer(cin, 64, 1, "f32", w, H, W)
    wins = [_window(rng, n, cin, H, W, fscale, "f32") for n in (500, 200)]
    for idx, f in wins:
        f *= np.exp2(rng.integers(-8, 9, (len(idx), 1))).astype(np.float32)  # and pillars
    for win in wins:
        _step(eng, win, "f32", True)
    _check(eng, wins, w, cin, 1, "f32", H, W, f"cin {cin} features {fscale} weights {wscale}")


@pytest.mark.parametrize("cin", [16, 64, 128])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_values_that_are_not_finite(cin, value):
    """An infinity or a NaN in one pillar reaches every output under it and no
    other."""
    H, W = 37, 41
    rng = np.random.default_rng(cin)
    w = rng.standard_normal((64, cin, 3, 3)).astype(np.float32)
    eng = _layer(cin, 64, 1, "f32", w, H, W)
    idx, f = _window(rng, 600, cin, H, W, 1.0, "f32")
    at = 300
    f[at, cin // 2] = value
    _step(eng, (idx, f), "f32", True)
    out = eng.read(1)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    r, c = divmod(int(idx[at]), W)
    under = np.zeros((H, W), bool)
    under[max(r - 1, 0):r + 2, max(c - 1, 0):c + 2] = True
    assert not np.isfinite(got[under]).any()
    f[at, cin // 2] = 0.0
    ref = _conv(_canvas((idx, f), cin, H, W), w, 1)
    np.testing.assert_allclose(got[~under], ref[~under], rtol=0, atol=1e-5 * np.abs(ref).max())


def test_first_pass_of_neck_inputs_of_16_and_32_channels():
    """Upsamplers read delta rows of fewer than 32 channels too."""
    from paper_2512_08557_amd import Engine
    rng = np.random.default_rng(5)
    H, W = 40, 48
    layers = [(16, 16, 2, True), (16, 32, 2, True)]
    ws = [(rng.standard_normal((co, ci, 3, 3)) * (2.0 / (9 * ci)) ** 0.5).astype(np.float32) for ci, co, _s, _r in layers]
    ups = [(1, 16, 1, True), (2, 32, 2, True)]
    us = [(rng.standard_normal((layers[u[0] - 1][1], u[1], u[2], u[2])) * 0.3).astype(np.float32) for u in ups]
    eng = Engine(H, W, 16, layers, ws, max_pillars=H * W, ups=ups, up_weights=us)
    for n in (500, 300):
        win = _window(rng, n, 16, H, W, 1.0, "f32")
        _step(eng, win, "f32", True)
    ys = oracle.forward(_canvas(win, 16, H, W), ws, layers)
    ref = oracle.forward_neck(ys, us, ups)
    out = eng.read(3)
    torch.cuda.synchronize()
    # three layers in a chain, each off by at most about 2e-6 of its largest sum
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=0, atol=6e-6 * np.abs(ref).max())
