"""The closure scan fused into the hashing pass over contents that the ordinary
ones do not hold: zeros and small integers under windows that reach below
4 GiB, and memory full of out-of-range pointers, for every kind of hash unit,
against the oracle (whole numbers: no tolerance).  The time of a pass must not
depend on such contents: it is held against the same pass over plain ones.

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE = 4096
CAP = 50


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


def check_scans(kc, ctx, ranges, views, unit, win):
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    expect = oracle.closure_scan(ranges, views, win_lo=win[0], win_hi=win[1], oob_cap=CAP)
    scan = kc.ScanOut("cuda", CAP, *win)
    kc.page_hash(ctx, rs, scan=scan)
    assert scan.result() == expect
    scan = kc.ScanOut("cuda", CAP, *win)
    kc.snapshot(ctx, rs, scan=scan)
    assert scan.result() == expect
    rs.close()


def large(total=512 << 20, n=48):
    """48 ranges of one buffer, and the buffer's words."""
    buf = torch.zeros(total + PAGE, dtype=torch.uint8, device="cuda")
    base = -(-buf.data_ptr() // PAGE) * PAGE
    step = total // n // PAGE * PAGE
    return buf, [(base + i * step, step - PAGE) for i in range(n)]


@pytest.mark.parametrize("unit", [PAGE, 4 * PAGE, 16 * PAGE])
def test_windows_below_4gib(kc, unit):
    rng = np.random.default_rng(unit)
    sizes = rng.integers(1, 60, size=30) * PAGE - rng.integers(0, PAGE, size=30)
    lay = W.make_layout(rng, sizes, gap_pages=(1, 3))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = np.zeros(lay.arena_bytes, dtype=np.uint8)
    words = host[: lay.arena_bytes // 8 * 8].view(np.uint64)
    at = rng.random(len(words))
    words[at < 0.5] = rng.integers(1, 9000, size=int((at < 0.5).sum()), dtype=np.uint64)
    low = (at > 0.9) & (at < 0.93)
    words[low] = rng.integers(1 << 31, 1 << 33, size=int(low.sum()), dtype=np.uint64)
    words[at > 0.99] = np.array([ranges[i % 30][0] for i in range(int((at > 0.99).sum()))], dtype=np.uint64)
    words[at > 0.999] = np.uint64(2**64 - 1)
    arena.buf.copy_(torch.from_numpy(host))
    views = W.host_views(lay, host)
    ctx = kc.Context(0)
    for win in ((1, 2**64 - 1), (4096, 1 << 47), (4096, 4097), (5000, (1 << 32) + 7), (1 << 32, 1 << 47), (0, 0)):
        say(f"scan windows: unit {unit}, window {win[0]:#x} .. {win[1]:#x}")
        check_scans(kc, ctx, ranges, views, unit, win)
    ctx.close()


def test_windows_below_4gib_time(kc):
    say("scan windows: time over zeros, window from 4096")
    buf, ranges = large()
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    us = {}
    for name, win in (("default", (0, 0)), ("low", (4096, 1 << 47))):
        scan = kc.ScanOut("cuda", CAP, *win)
        out = kc.page_hash(ctx, rs, scan=scan)
        us[name] = best_us(lambda: kc.page_hash(ctx, rs, scan=scan, out=out))
    say(f"scan windows: {us}")
    assert us["low"] < 1.25 * us["default"]
    rs.close()
    ctx.close()


@pytest.mark.parametrize("unit", [PAGE, 2 * PAGE, 8 * PAGE, 16 * PAGE, 64 * PAGE, 512 * PAGE])
def test_memory_of_out_of_range_words(kc, unit):
    """Every word, every word of some pages, and a few words are pointers past
    the end of a range."""
    rng = np.random.default_rng(7 + unit)
    sizes = np.concatenate([rng.integers(1, 5, size=6) * unit, rng.integers(1, 40, size=12) * PAGE])
    sizes -= rng.integers(0, PAGE, size=len(sizes))
    lay = W.make_layout(rng, sizes, gap_pages=(1, 3))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    words_of = lay.arena_bytes // 8
    past = np.array([b + s + 8 for b, s in ranges], dtype=np.uint64)[rng.integers(0, len(ranges), size=words_of)]
    inside = np.array([b for b, _ in ranges], dtype=np.uint64)[rng.integers(0, len(ranges), size=words_of)]
    ctx = kc.Context(0)
    for name, share in (("every word", np.ones(words_of, dtype=bool)),
                        ("every word of a third of the pages", (rng.random(words_of // 512 + 1) < 0.33).repeat(512)[:words_of]),
                        ("one word in 50", rng.random(words_of) < 0.02)):
        say(f"out-of-range words: unit {unit}, {name}")
        host = np.zeros(lay.arena_bytes, dtype=np.uint8)
        host[: words_of * 8].view(np.uint64)[:] = np.where(share, past, np.where(rng.random(words_of) < 0.1, inside, 5))
        arena.buf.copy_(torch.from_numpy(host))
        check_scans(kc, ctx, ranges, W.host_views(lay, host), unit, (0, 0))
    ctx.close()


@pytest.mark.parametrize("unit", [PAGE, 16 * PAGE])
def test_memory_of_out_of_range_words_time(kc, unit):
    buf, ranges = large()
    words = buf[: buf.numel() // 8 * 8].view(torch.int64)
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    us = {}
    for name, value in (("in range", ranges[3][0] + 64), ("out of range", ranges[3][0] + ranges[3][1] + 64)):
        say(f"out-of-range words: time, unit {unit}, all words {name}")
        words.fill_(value)
        scan = kc.ScanOut("cuda", CAP)
        out = kc.page_hash(ctx, rs, scan=scan)
        us[name] = best_us(lambda: kc.page_hash(ctx, rs, scan=scan, out=out))
    say(f"out-of-range words: {us}")
    assert us["out of range"] < 2.0 * us["in range"]
    rs.close()
    ctx.close()
