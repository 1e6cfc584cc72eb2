"""Change lists built by stream compaction (every layer after the first): grid
widths around the 32-cell words, rows of one word and of more than a tile's
words, single rows and columns, both strides, batches, sparse and full change
sets; and very large grids, whose lists come from the layers' tiles.  The
lists, pair counts and maps are checked against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import note

pytestmark = pytest.mark.gpu

CHAINS = {"s1s1": (1, 1, 1), "s2s2": (2, 2, 2), "s1s2s1": (1, 2, 1, 1)}


def _run(H, W, strides, fill, batch=1):
    from paper_2512_08557_amd import Engine
    rng = np.random.default_rng(H * 100003 + W * 7 + len(strides) + batch)
    layers = [(16, 16, s, True) for s in strides]
    ws = [(rng.standard_normal((16, 16, 3, 3)) / 12).astype(np.float32) for _ in layers]
    eng = Engine(H, W, 16, layers, ws, max_pillars=H * W * batch, batch=batch)
    cells = H * W * batch
    prev = np.zeros((batch, H, W, 16), np.uint32)
    x = np.zeros((cells, 16), np.float32)
    for step, f in enumerate((fill, 0.02, fill)):
        change = rng.random(cells) < f
        x = x.copy()
        x[change] = rng.standard_normal((int(change.sum()), 16)).astype(np.float32)
        idx = np.flatnonzero(np.any(x != 0, axis=1)).astype(np.int32)
        note(f"[gpu-test] plan {H}x{W}x{batch} {strides} step {step}: {len(idx)} pillars")
        eng.step(torch.from_numpy(idx).cuda(), torch.from_numpy(x[idx]).cuda(), sorted=True)
        canvas = x.reshape(batch, H, W, 16)
        bits = np.ascontiguousarray(canvas).view(np.uint32)
        want = None
        pairs = np.zeros(len(layers) + 1, np.int64)
        for b in range(batch):
            lists = oracle.changed_lists(prev[b], bits[b], list(strides))
            m = np.isin(np.arange(H * W), lists[0]).reshape(H, W)
            h, w = H, W
            for l, s in enumerate(strides, 1):
                pairs[l] += oracle.pair_counts(m, s)
                h, w = (h - 1) // s + 1, (w - 1) // s + 1
                m = np.isin(np.arange(h * w), lists[l]).reshape(h, w)
            off = [H * W * b]
            h, w = H, W
            for s in strides:
                h, w = (h - 1) // s + 1, (w - 1) // s + 1
                off.append(h * w * b)
            lists = [a + o for a, o in zip(lists, off)]
            want = lists if want is None else [np.concatenate([p, q]) for p, q in zip(want, lists)]
        for l, ref in enumerate(want):
            np.testing.assert_array_equal(eng.changed(l), ref, err_msg=f"A_{l}")
        dst = torch.empty(cells, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        eng.changed_noalloc(len(layers), dst, cnt)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(dst[:int(cnt)].cpu().numpy(), want[-1])
        assert eng.stats()["pairs"][1:] == list(pairs[1:])
        prev = bits
    for l in range(1, len(layers) + 1):
        out = eng.read(l)
        torch.cuda.synchronize()
        got = out.cpu().numpy().reshape((batch,) + eng.shapes[l])
        for b in range(batch):
            ref = oracle.forward(canvas[b].astype(np.float64), ws, layers)[l - 1]
            # a few short sums in a chain, three strides: each off by about 2e-7 of its largest
            np.testing.assert_allclose(got[b], ref, rtol=0, atol=5e-6 * max(np.abs(ref).max(), 1e-3))


@pytest.mark.parametrize("chain", sorted(CHAINS))
@pytest.mark.parametrize("W", [1, 2, 31, 32, 33, 63, 64, 65, 130])
@pytest.mark.parametrize("fill", [0.01, 1.0])
def test_row_widths(W, chain, fill):
    _run(23, W, CHAINS[chain], fill)


@pytest.mark.parametrize("H,W", [(1, 1), (1, 200), (200, 1), (3, 4097), (5, 9001), (301, 70)])
@pytest.mark.parametrize("chain", ["s1s1", "s1s2s1"])
def test_grid_shapes(H, W, chain):
    _run(H, W, CHAINS[chain], 0.05)


@pytest.mark.parametrize("chain", sorted(CHAINS))
def test_batches(chain):
    _run(37, 45, CHAINS[chain], 0.05, batch=3)


@pytest.mark.parametrize("W,batch", [(2, 4), (2, 5), (33, 3)])
@pytest.mark.parametrize("chain", ["s1s1", "s1s2s1"])
def test_grids_on_either_side_of_the_rule(W, batch, chain):
    """2^17 words of 32 cells (a row has one at least) is the largest grid whose
    lists are compacted: 4 x 32767 rows of one word are just below, 5 x 32767 and
    3 x 32767 rows of two above (in the layers before stride 2)."""
    _run(32767, W, CHAINS[chain], 0.002, batch=batch)


def test_a_stride_of_a_large_grid_takes_the_time_of_its_changes():
    """Twenty changed pillars on 4096x4096: a compaction of the whole grid per
    layer took 48 us a stride (58 with the bitmap's clear), the tiles' footprint
    23."""
    from paper_2512_08557_amd import Engine
    H = W = 4096
    rng = np.random.default_rng(0)
    ws = [(rng.standard_normal((16, 16, 3, 3)) / 12).astype(np.float32)] * 3
    eng = Engine(H, W, 16, [(16, 16, 1, True)] * 3, ws, max_pillars=64)
    idx = torch.from_numpy(np.sort(rng.choice(H * W, 20, replace=False)).astype(np.int32)).cuda()
    f = [torch.from_numpy(rng.standard_normal((20, 16)).astype(np.float32)).cuda() for _ in range(2)]
    for k in range(6):
        eng.step(idx, f[k & 1], sorted=True)
    eng.profile(True)
    for k in range(20):
        eng.step(idx, f[k & 1], sorted=True)
    ms, _cnt = eng.profile_read()
    eng.profile(False)
    assert sum(ms) / 20 < 0.040, f"{1e3 * sum(ms) / 20:.1f} us of kernels per stride"


def test_a_small_grid_is_cut_into_several_tiles():
    """Two 16-channel layers on 64x64 whose launches also build the next list,
    and one that does not.  One workgroup over the whole grid took 7.0 us beside
    the last layer's 4.1; four take 4.8."""
    from paper_2512_08557_amd import Engine
    rng = np.random.default_rng(0)
    ws = [(rng.standard_normal((16, 16, 3, 3)) / 12).astype(np.float32)] * 3
    eng = Engine(64, 64, 16, [(16, 16, 1, True)] * 3, ws, max_pillars=400)
    idx = torch.from_numpy(np.sort(rng.choice(64 * 64, 400, replace=False)).astype(np.int32)).cuda()
    f = [torch.from_numpy(rng.standard_normal((400, 16)).astype(np.float32)).cuda() for _ in range(2)]
    for k in range(10):
        eng.step(idx, f[k & 1], sorted=True)
    eng.profile(True)
    for k in range(50):
        eng.step(idx, f[k & 1], sorted=True)
    ms, _cnt = eng.profile_read()
    assert ms[2] + ms[3] < 2 * 1.4 * ms[4], [f"{m / 50 * 1e3:.2f} us" for m in ms]
