"""The compare over contents that ordinary outputs do not hold: buffers that are
NaN all over or in long stretches, in one side or in both, with equal and with
other payloads, against the oracle (integers and exact fp64 maxima: no
tolerance).  The time of a pass over them is held against the pass over other
contents of the same buffers.

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
FLOATS = sorted(d for d, t in W.TORCH_DTYPE.items() if t.is_floating_point)


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def best_us(fn, reps=5):
    """Shortest time of a call among some, after one that is not timed."""
    fn()
    ms = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms) * 1e3


def nan_codes(dt):
    """Two NaN encodings of a type as bytes (formats with one: it twice)."""
    t = W.TORCH_DTYPE[dt]
    if "fnuz" in str(t):
        return b"\x80", b"\x80"
    if dt == W.DT_FP8:
        return b"\x7f", b"\xff"
    return {1: (b"\x7d", b"\xfe"), 2: (b"\xc1\x7f", b"\x02\xff"), 4: (b"\x01\x00\xc0\x7f", b"\x00\x01\x80\xff"),
            8: (b"\x01" + b"\x00" * 5 + b"\xf0\x7f", b"\x00\x00\x00\x00\x01\x00\xf0\xff")}[W.ELEM_SIZE[dt]]


def check(kc, host, dt, name):
    """All pairs of (candidate, golden) host bytes in one call of each kind."""
    say(f"compare contents: dtype {dt}, {name}")
    dev = [tuple(torch.from_numpy(x).cuda() for x in p) for p in host]
    pairs = [(c, g, dt, 3, 1e-3, 1e-2) for c, g in dev]
    expect = [oracle.compare(c, g, dt, 3, 1e-3, 1e-2) for c, g in host]
    ctx = kc.Context(0)
    for tile in (0, 16384):
        ctx.set_tuning(kc.OP_COMPARE, tile_bytes=tile)
        assert kc.decode_cmp(kc.compare(ctx, pairs), len(pairs)) == expect
        for p, e in zip(pairs, expect):  # alone: small ones take the report of the pass
            assert kc.decode_cmp(kc.compare(ctx, [p]), 1) == [e]
    ctx.close()


@pytest.mark.parametrize("dt", FLOATS)
def test_nan_filled(kc, dt):
    rng = np.random.default_rng(dt)
    w = W.ELEM_SIZE[dt]
    one, two = (np.frombuffer(c, dtype=np.uint8) for c in nan_codes(dt))
    host = []
    for n in (1, 16 // w + 1, 1000, 16384 // w + 3, 70000 // w, 200001 // w):
        plain = torch.from_numpy(rng.standard_normal(n)).to(W.TORCH_DTYPE[dt]).view(torch.uint8).numpy().copy()
        full, other = np.tile(one, n), np.tile(two, n)
        mixed = plain.copy().reshape(n, w)
        mixed[rng.random(n) < 0.5] = one
        stretch = plain.copy().reshape(n, w)
        stretch[n // 3:n // 2 + 1] = two
        moved = plain.copy().reshape(n, w)
        moved[rng.random(n) < 0.2, 0] ^= 1
        mixed, stretch, moved = mixed.reshape(-1), stretch.reshape(-1), moved.reshape(-1)
        host += [(full, full.copy()), (full, other), (full, plain), (plain, full), (mixed, plain), (plain, mixed),
                 (mixed, mixed.copy()), (mixed, stretch), (stretch, stretch.copy()), (moved, stretch)]
    check(kc, host, dt, "NaN all over, in half of the elements, in a stretch")


@pytest.mark.parametrize("dt", FLOATS)
def test_few_nans(kc, dt):
    """NaNs as a thread of the pass meets them: k of its 16-byte runs' elements
    (four runs, 256 * 16 bytes apart) for k around the number from which a wave
    counts them together, in few or all threads, among elements that differ; then
    scattered ones."""
    rng = np.random.default_rng(100 + dt)
    w = W.ELEM_SIZE[dt]
    per = 16 // w
    one, two = (np.frombuffer(c, dtype=np.uint8) for c in nan_codes(dt))
    n = 2 * 16384 // w + 5 * per + 3  # two rounds of a workgroup, some runs and a tail
    host = []

    def add(at, first, second, off):
        gold = torch.from_numpy(rng.standard_normal(n)).to(W.TORCH_DTYPE[dt]).view(torch.uint8).numpy().copy().reshape(n, w)
        cand = gold.copy()
        cand[rng.random(n) < off, 0] ^= 1
        for side, code in ((cand, first), (gold, second)):
            if code is not None:
                side[at] = code
        host.append((cand.reshape(-1), gold.reshape(-1)))

    for k in sorted({1, 2, min(11, 4 * per), min(12, 4 * per), min(13, 4 * per), 4 * per}):
        for threads in ([5], [0, 63, 64, 200, 255], range(256)):
            of_thread = [rng.permutation(4 * per)[:k] for _ in threads]
            at = np.concatenate([(t + 256 * (e // per)) * per + e % per for t, e in zip(threads, of_thread)])
            add(at, one, None, 0.1)
            add(at, one, one, 0.0)
            add(at, two, one, 0.5)
    for p in (1e-3, 0.01, 0.1):
        at = np.flatnonzero(rng.random(n) < p)
        add(at, one, two, 0.113)
        add(at, None, two, 0.0)
    check(kc, host, dt, "few NaNs")


@pytest.mark.parametrize("dt", [d for d in FLOATS if W.ELEM_SIZE[d] < 8])
def test_nan_filled_time(kc, dt):
    """A pass over NaNs is no longer than over elements that all differ."""
    n = (128 << 20) // W.ELEM_SIZE[dt]
    raw = torch.randint(0, 100, (n * W.ELEM_SIZE[dt],), dtype=torch.uint8, device="cuda")
    other = raw ^ 1
    nan = torch.from_numpy(np.frombuffer(nan_codes(dt)[0], dtype=np.uint8).copy()).cuda().repeat(n)
    ctx = kc.Context(0)
    us = {}
    for name, c, g in (("all off", other, raw), ("NaN in both", nan, nan.clone()), ("NaN in one", nan, raw)):
        say(f"compare contents: time, dtype {dt}, {name}")
        ps = kc.PairSet(ctx, [(c, g, dt, 3, 1e-3, 1e-2)])
        res = kc.compare_pairset(ctx, ps)
        us[name] = best_us(lambda: kc.compare_pairset(ctx, ps, res))
        ps.close()
    say(f"compare contents: {us}")
    assert us["NaN in both"] < 1.25 * us["all off"]
    assert us["NaN in one"] < 1.25 * us["all off"]
    ctx.close()


def test_raw_bytes(kc):
    """One differing byte at every place of a run, of a few runs and past the
    last one, then all and half of them."""
    rng = np.random.default_rng(9)
    host = []
    for n in (7, 300, 5000, 40000, 150001):
        gold = rng.integers(0, 256, size=n, dtype=np.uint8)
        spots = [[i] for i in list(range(min(n, 70))) + [n - 1, n // 2]]
        spots += [rng.integers(0, n, size=3) for _ in range(4)] + [np.flatnonzero(rng.random(n) < 0.5), np.arange(n)]
        for at in spots:
            cand = gold.copy()
            cand[at] ^= rng.integers(1, 256, size=len(at)).astype(np.uint8)
            host.append((cand, gold))
    check(kc, host, W.DT_U8, "raw bytes that differ at every place")


def test_raw_bytes_time(kc):
    """Raw bytes that all differ cost little more than equal ones."""
    gold = torch.randint(0, 256, (128 << 20,), dtype=torch.uint8, device="cuda")
    ctx = kc.Context(0)
    us = {}
    for name, cand in (("equal", gold.clone()), ("all off", gold ^ 3)):
        say(f"compare contents: time, raw bytes, {name}")
        ps = kc.PairSet(ctx, [(cand, gold, W.DT_U8, 0)])
        res = kc.compare_pairset(ctx, ps)
        us[name] = best_us(lambda: kc.compare_pairset(ctx, ps, res))
        ps.close()
    say(f"compare contents: {us}")
    assert us["all off"] < 2.0 * us["equal"]
    ctx.close()
