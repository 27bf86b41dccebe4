"""The compare's exact path where rounds, tiles and workgroups end: lengths
around one round of a workgroup (16 KiB a side) and around a tile, from one
differing element to all of them, NaNs in either side, aligned and shifted
buffers, ties and underflows of the relative error.  Every report equals the
oracle's (integers and exact fp64 maxima: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
ROUND = 16384   # bytes of each side a workgroup takes per round


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def _bytes_pair(rng, dt, n, density, nans):
    """Host bytes of a golden and a candidate: N(0, 1) values (integers:
    uniform), `density` of the elements with their low bits changed."""
    w = W.ELEM_SIZE[dt]
    t = W.TORCH_DTYPE[dt]
    if t.is_floating_point:
        gold = torch.from_numpy(rng.standard_normal(n)).to(t).view(torch.uint8).numpy().copy()
    else:
        gold = rng.integers(0, 256, size=n * w, dtype=np.uint8)
    cand = gold.copy()
    hit = np.flatnonzero(rng.random(n) < density)
    if density and len(hit) == 0:
        hit = rng.integers(0, n, size=1)
    cand.reshape(n, w)[hit, 0] ^= rng.integers(1, 4, size=len(hit)).astype(np.uint8)
    if nans and t.is_floating_point:
        code = np.frombuffer({1: b"\x80" if "fnuz" in str(t) else b"\x7f", 2: b"\xc1\x7f", 4: b"\x01\x00\xc0\x7f",
                              8: b"\x01\x00\x00\x00\x00\x00\xf8\x7f"}[w], dtype=np.uint8)
        for side in ((gold, cand), (gold,), (cand,)):
            at = rng.integers(0, n, size=max(1, n // 500))
            for s in side:
                s.reshape(n, w)[at] = code
    return gold, cand


@pytest.mark.parametrize("dt", sorted(W.TORCH_DTYPE))
def test_rounds_tiles_and_densities(kc, dt):
    say(f"compare rounds: dtype={dt}, lengths around rounds and tiles, one to all elements differing")
    rng = np.random.default_rng(100 + dt)
    w = W.ELEM_SIZE[dt]
    lengths = [1, 16 // w + 1, ROUND // w - 1, ROUND // w, ROUND // w + 1, 4 * ROUND // w + 16 // w - 1, 9 * ROUND // w]
    host, pairs = [], []
    for i, n in enumerate(lengths):
        for density, nans, shift in ((0.0, False, 0), (1e-5, False, 1), (0.1, True, 0), (0.1, True, 3), (1.0, False, 0)):
            gold, cand = _bytes_pair(rng, dt, n, density, nans)
            dev = []
            for b in (cand, gold):
                buf = torch.full((n * w + shift * w + 64,), 0x5A, dtype=torch.uint8, device="cuda")
                buf[shift * w: shift * w + n * w] = torch.from_numpy(b).cuda()
                dev.append(buf[shift * w: shift * w + n * w])
            host.append((cand, gold))
            pairs.append((dev[0], dev[1], dt, i % 4, 1e-3, 1e-2))
    want = [oracle.compare(c, g, dt, p[3], p[4], p[5]) for (c, g), p in zip(host, pairs)]
    for grid, tile in ((0, 0), (1, 4096), (1024, 65536)):
        ctx = kc.Context(0)
        ctx.set_tuning(kc.OP_COMPARE, grid_per_cu=grid, tile_bytes=tile)
        assert kc.decode_cmp(kc.compare(ctx, pairs), len(pairs)) == want, (grid, tile)
        ps = kc.PairSet(ctx, pairs)
        for _ in range(2):   # the accumulators are clear again after a call
            assert kc.decode_cmp(kc.compare_pairset(ctx, ps), len(pairs)) == want, (grid, tile)
        res = torch.zeros(len(pairs) * kc.RESULT_BYTES, dtype=torch.uint8, device="cuda")
        assert kc.decode_cmp(kc.compare_noalloc(ctx, pairs, res), len(pairs)) == want, (grid, tile)
        ps.close()
        ctx.close()


@pytest.mark.parametrize("dt", [W.DT_F64, W.DT_F32, W.DT_BF16, W.DT_F16, W.DT_FP8, W.DT_FP8_E5M2])
def test_relative_error_ties_and_extremes(kc, dt):
    """The relative error grows, ties and underflows: random codes of the whole
    encoding (subnormals, infinities, NaNs, zeros of both signs)."""
    say(f"compare relative error: dtype={dt}, random codes")
    rng = np.random.default_rng(7 + dt)
    n = 40000
    w = W.ELEM_SIZE[dt]
    gold = rng.integers(0, 256, size=n * w, dtype=np.uint8)
    cand = rng.integers(0, 256, size=n * w, dtype=np.uint8)
    g64 = np.zeros(n * w, dtype=np.uint8)
    if dt == W.DT_F64:   # subnormal errors over normal and subnormal golds
        g64.view("<u8")[:] = rng.integers(1, 1 << 53, size=n, dtype=np.uint64)
    c64 = g64.copy()
    c64.reshape(n, w)[:, 0] ^= 1
    pairs = [(cand, gold), (gold, cand), (c64, g64), (cand, g64)]
    dev = [(torch.from_numpy(c).cuda(), torch.from_numpy(g).cuda(), dt, 0, 0.0, 1e-3) for c, g in pairs]
    ctx = kc.Context(0)
    got = kc.decode_cmp(kc.compare(ctx, dev), len(dev))
    for r, (c, g) in zip(got, pairs):
        assert r == oracle.compare(c, g, dt, 0, 0.0, 1e-3)
    ctx.close()
