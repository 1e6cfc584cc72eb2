"""Single layers at the sizes where the layer kernel's tiling and its split
fp32 operands can go wrong: list lengths around whole tiles, every channel
count, both strides, values far from 1, output and input channels of scales far
apart, single products, and values that are not finite or nearly so."""
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
    sum of K = 9*cin products to every touched cell.  fp32: the three planes
    hold a value exactly, h within 2^-8 of it and h + m within 2^-17, so
    the products left out (m*l, l*m, l*l) are at most 2^-24 + 2^-34 of the whole;
    summing takes at most three roundings per channel unit (its large products,
    its small ones, their sum) and one per wavefront and for Z (16 in all), 2^-24
    each of the sum of magnitudes.  bf16 products are exact, and the output is
    rounded to bf16."""
    units = 9 * max(1, cin // 32)
    eps = (0 if dtype == "bf16" else 2.0 ** -24 + 2.0 ** -34) + (3 * units + 16) * 2.0 ** -24
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c", [32, 64, 128, 256])
@pytest.mark.parametrize("k", [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 2047, 2048, 2049, 2063, 2064, 2065, 2079, 2080])
def test_segment_lengths_around_tiles(k, c, dtype):
    """A list's two segments of exactly k entries each: pillars that change one
    cell of either layer each (stride 2, even positions), in pairs side by side,
    so that every tile of the compaction, which gives either segment half of its
    cells, holds an even number.  Up to 64 channels, and in fp32 always, lists of
    up to 2048 entries a segment (16 for each of 128 workgroups) take 16-cell
    tiles, longer ones 32; wider bf16 layers take 32-cell tiles throughout."""
    from paper_2512_08557_amd import Engine
    G = 32 if k < 512 else 96                               # the second layer's grid, G x G
    H = W = 4 * G
    rng = np.random.default_rng(c + k)
    ws = [(rng.standard_normal((co, ci, 3, 3)) * (2.0 / (9 * ci)) ** 0.5).astype(np.float32)
          for ci, co in ((16, c), (c, 32))]
    if dtype == "bf16":
        ws = [_bf16(w) for w in ws]
    layers = [(16, c, 2, True), (c, 32, 2, False)]
    eng = Engine(H, W, 16, layers, ws, dtype=dtype, max_pillars=H * W)
    pair = rng.choice(G * G // 2, k, replace=False)
    pos = np.concatenate([2 * pair, 2 * pair + 1])          # cells of the second layer's grid
    idx = np.sort(pos // G * 4 * W + pos % G * 4).astype(np.int32)
    f = rng.standard_normal((2 * k, 16)).astype(np.float32)
    if dtype == "bf16":
        f = _bf16(f)
    note(f"[gpu-test] segments of {k}, {c} channels {dtype}")
    _step(eng, (idx, f), dtype, True)
    assert len(eng.changed(1)) == len(eng.changed(2)) == 2 * k
    ys = oracle.forward(_canvas((idx, f), 16, H, W), ws, layers, bf16_storage=dtype == "bf16")
    out = eng.read(2)
    torch.cuda.synchronize()
    got, ref = out.float().cpu().numpy().astype(np.float64), ys[1]
    # two layers of one tap each; bf16 rounds the first one's outputs and its own
    tol = 1e-6 if dtype == "f32" else 2.0 ** -7
    assert np.abs(got - ref).max(initial=0) <= tol * max(np.abs(ref).max(initial=0), 1e-30)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout", [(64, 64), (128, 8), (128, 128), (256, 256)])
def test_lists_on_either_side_of_the_tile_height(cin, cout, dtype):
    """Lists somewhat shorter and longer than what 16-cell tiles take, for one to
    four groups of 64 output channels (256 workgroups walk two segments of each)."""
    H, W = 200, 200
    rng = np.random.default_rng(cin + cout)
    w = (rng.standard_normal((cout, cin, 3, 3)) * (2.0 / (9 * cin)) ** 0.5).astype(np.float32)
    if dtype == "bf16":
        w = _bf16(w)
    most = 2 * 16 * (256 // (2 * max(1, cout // 64)))
    eng = _layer(cin, cout, 1, dtype, w, H, W)
    wins = []
    for rows in (most * 3 // 4 // W, most * 5 // 4 // W + 1):   # of changed cells, and one more in the list
        f = rng.standard_normal((rows * W, cin)).astype(np.float32)
        wins.append((np.arange(rows * W, dtype=np.int32), _bf16(f) if dtype == "bf16" else f))
    for win, longer in zip(wins, (False, True)):
        _step(eng, win, dtype, True)
        n = len(eng.changed(1))
        # (the two segments of a detected list differ by a workgroup's cells or so)
        assert n > most * 1.1 if longer else n < most * 0.95
    _check(eng, wins, w, cin, 1, dtype, H, W, f"{cin}->{cout} {dtype}")


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


def _unlike(rng, cin, spread):
    """2^0 .. 2^spread over the input channels, in any order."""
    return np.exp2(np.linspace(0, spread, cin) - spread / 2)[rng.permutation(cin)].astype(np.float32)


@pytest.mark.parametrize("cin", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("spread", [12, 24, 30, 60])
def test_input_channels_of_unlike_scale(cin, spread):
    """Features 2^spread apart between the channels of a unit, weights the other
    way round, so that every channel counts alike in the sums."""
    H, W = 37, 41
    rng = np.random.default_rng(cin + spread)
    s = _unlike(rng, cin, spread)
    w = (rng.standard_normal((32, cin, 3, 3)) / s[None, :, None, None]).astype(np.float32)
    eng = _layer(cin, 32, 1, "f32", w, H, W)
    wins = [_window(rng, n, cin, H, W, 1.0, "f32") for n in (500, 60)]
    for _idx, f in wins:
        f *= s
    for win in wins:
        _step(eng, win, "f32", True)
    _check(eng, wins, w, cin, 1, "f32", H, W, f"cin {cin} spread 2^{spread}")


@pytest.mark.parametrize("cin", [16, 64, 128])
@pytest.mark.parametrize("ratio", [1e5, 1e7, 1e9, 1e20])
def test_a_large_input_channel_of_weight_zero(cin, ratio):
    H, W = 37, 41
    rng = np.random.default_rng(cin)
    w = rng.standard_normal((32, cin, 3, 3)).astype(np.float32)
    w[:, 3] = 0.0
    w[5, 7] *= ratio                                        # and one large weight, of a channel that is zero
    eng = _layer(cin, 32, 1, "f32", w, H, W)
    wins = [_window(rng, n, cin, H, W, 1.0, "f32") for n in (500, 60)]
    for _idx, f in wins:
        f[:, 3] *= ratio
        f[:, 7] = 0.0
    for win in wins:
        _step(eng, win, "f32", True)
    _check(eng, wins, w, cin, 1, "f32", H, W, f"cin {cin} ratio {ratio}")


@pytest.mark.parametrize("cin", [16, 32, 128])
def test_single_products(cin):
    """One channel of one pillar under every output: what is read is one fp32
    product, off by the products left out and a few roundings."""
    H, W = 37, 41
    rng = np.random.default_rng(cin)
    w = rng.standard_normal((64, cin, 3, 3)).astype(np.float32)
    eng = _layer(cin, 64, 1, "f32", w, H, W)
    idx = np.array([(r * W + c) for r in range(1, H, 3) for c in range(1, W, 3)], np.int32)
    f = np.zeros((len(idx), cin), np.float32)
    f[np.arange(len(idx)), rng.integers(0, cin, len(idx))] = rng.standard_normal(len(idx))
    _step(eng, (idx, f), "f32", True)
    out = eng.read(1)
    torch.cuda.synchronize()
    got, ref = out.cpu().numpy().astype(np.float64), _conv(_canvas((idx, f), cin, H, W), w, 1)
    assert np.all(np.abs(got - ref) <= 3 * 2.0 ** -24 * np.abs(ref))


@pytest.mark.parametrize("cin", [16, 64, 128])
@pytest.mark.parametrize("fmax,wscale", [(3.4028235e38, 1e-4), (3.0e38, 1e-30), (1e33, 1.0), (1e-37, 1.0), (1e-36, 1e30)])
def test_ends_of_the_range(cin, fmax, wscale):
    """Features up to the largest float (which rounds to infinity in bf16) and
    down to the smallest normal ones: sums that fp32 holds stay finite."""
    H, W = 37, 41
    rng = np.random.default_rng(cin)
    w = (rng.standard_normal((32, cin, 3, 3)) * wscale / (9 * cin)).astype(np.float32)
    eng = _layer(cin, 32, 1, "f32", w, H, W)
    idx, f = _window(rng, 500, cin, H, W, 1.0, "f32")
    f = np.clip(f, -1, 1) * np.float32(fmax)                # many are exactly +-fmax
    _step(eng, (idx, f), "f32", True)
    # planes end at 2^-133 and products at 2^-149
    ref = _conv(_canvas((idx, f), cin, H, W), w, 1)
    mag = _conv(np.abs(_canvas((idx, f), cin, H, W)), np.abs(w), 1)
    tiny = 9 * cin * (2.0 ** -133 * np.abs(w).max() + 2.0 ** -133 * fmax * (wscale < 1e-20) + 2.0 ** -149)
    out = eng.read(1)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    eps = 2.0 ** -24 + 2.0 ** -34 + (3 * 9 * max(1, cin // 32) + 16) * 2.0 ** -24
    assert np.all(np.abs(got - ref) <= eps * mag + tiny)


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
    if np.isinf(value):                                     # infinite, with the weight's sign
        sign = np.sign(value) * np.sign(w[:, cin // 2])
        for i in range(max(r - 1, 0), min(r + 2, H)):
            for j in range(max(c - 1, 0), min(c + 2, W)):
                np.testing.assert_array_equal(got[i, j], np.inf * sign[:, r - i + 1, c - j + 1])
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


@pytest.mark.parametrize("cin,cout,s", [(16, 16, 1), (16, 32, 2), (32, 32, 2), (64, 64, 1), (128, 128, 2), (256, 64, 4)])
def test_upsampler_of_unlike_channels(cin, cout, s):
    """An upsampler behind a layer that passes its input on: channels 2^60 apart
    with weights the other way round, then an infinity and a value that rounds
    to one in bf16."""
    from paper_2512_08557_amd import Engine
    H, W = 21, 19
    rng = np.random.default_rng(cin + s)
    same = np.zeros((cin, cin, 3, 3), np.float32)
    same[np.arange(cin), np.arange(cin), 1, 1] = 1.0
    sc = _unlike(rng, cin, 60)
    u = (rng.standard_normal((cin, cout, s, s)) / sc[:, None, None, None]).astype(np.float32)
    eng = Engine(H, W, cin, [(cin, cin, 1, False)], [same], max_pillars=H * W, ups=[(1, cout, s, False)], up_weights=[u])
    idx, f = _window(rng, 150, cin, H, W, 1.0, "f32")
    f *= sc
    _step(eng, (idx, f), "f32", True)
    out = eng.read(2)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)

    def up(x, w):
        return np.einsum("hwc,cdab->hawbd", x, w.astype(np.float64)).reshape(H * s, W * s, cout)

    x = _canvas((idx, f), cin, H, W)
    eps = 2.0 ** -24 + 2.0 ** -34 + (3 * max(1, cin // 32) + 2) * 2.0 ** -24
    tol = eps * up(np.abs(x), np.abs(u))
    assert np.all(np.abs(got - up(x, u)) <= tol)
    # the next window, with special values in two pillars
    g = f.copy()
    inf_at, big_at = 40, 90
    g[inf_at, 3] = np.inf
    g[big_at, np.argmax(sc)] = 3.4028235e38                 # the channel with the smallest weights
    _step(eng, (idx, g), "f32", True)
    out = eng.read(2)
    torch.cuda.synchronize()
    got2 = out.cpu().numpy().astype(np.float64)
    r, c = divmod(int(idx[inf_at]), W)
    # (the layer's zero weights make NaNs of the infinity in its other channels
    # and in the cells around it)
    assert not np.isfinite(got2[r * s:r * s + s, c * s:c * s + s]).any()
    g[inf_at] = 0.0
    y = _canvas((idx, g), cin, H, W)
    want = up(y, u)
    # a stride adds what changed: the sums of both windows count
    tol = tol + eps * up(np.abs(x) + np.abs(y), np.abs(u))
    ok = np.ones((H * s, W * s), bool)
    ok[max(r - 1, 0) * s:(r + 2) * s, max(c - 1, 0) * s:(c + 2) * s] = False
    assert np.all((np.abs(got2 - want) <= tol)[ok])
    same_cells = ok.copy()
    r, c = divmod(int(idx[big_at]), W)
    same_cells[r * s:r * s + s, c * s:c * s + s] = False
    np.testing.assert_array_equal(got2[same_cells], got[same_cells])
