"""The hashing pass under everything that selects code or shapes it: 4, 8 and 16
units per wave (few, some and many tiles), one and four waves per workgroup,
the built-in grid and tuned ones whose waves stride over the tiles, one launch
per range, with a scan of either kind of window and with a prior table, pages
and larger units, all against the oracle and so against each other (whole
numbers and bytes: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE, KiB, MiB = 4096, 1 << 10, 1 << 20
SHAPES = (dict(), dict(grid_per_cu=1), dict(grid_per_cu=3), dict(grid_per_cu=24), dict(per_item=1), dict(per_item=1, grid_per_cu=2))


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


# ranges, units per range at most, unit: few, some and many tiles of each
@pytest.mark.parametrize("n_ranges,most,unit", [(20, 30, PAGE), (200, 40, PAGE), (1500, 20, PAGE), (40, 20, 16 * KiB),
                                                (700, 9, 16 * KiB), (2300, 2, 16 * KiB), (30, 9, 64 * KiB), (9, 4, 2 * MiB)])
def test_shapes_agree(kc, n_ranges, most, unit):
    rng = np.random.default_rng(n_ranges * 3 + most + unit)
    sizes = rng.integers(1, most + 1, size=n_ranges) * unit
    sizes = sizes - np.where(rng.random(n_ranges) < 0.5, rng.choice([1, 8, 31, 33, 1000, 4064, 4095], size=n_ranges), 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(0, 256, size=lay.arena_bytes, dtype=np.uint8)
    words = host[: lay.arena_bytes // 8 * 8].view(np.uint64)
    at = rng.choice(len(words), size=max(8, len(words) // 200), replace=False)
    to = rng.integers(0, n_ranges, size=len(at))
    words[at] = np.array([ranges[i][0] + ranges[i][1] * (j % 3 == 0) for j, i in enumerate(to)], dtype=np.uint64)
    for i in np.flatnonzero(rng.random(lay.arena_bytes // unit + 1) < 0.25):
        host[i * unit:(i + 1) * unit] = 0
    arena.buf.copy_(torch.from_numpy(host))
    views = W.host_views(lay, host)
    oh, oz, _ = oracle.page_hash(ranges, views, seed=3, unit=unit)
    op, ova, onk = oracle.compact(ranges, views, oz, unit=unit)
    prior = oh.copy()
    prior[::5] ^= np.uint64(1)
    _, _, oc = oracle.page_hash(ranges, views, seed=3, prior=prior, unit=unit)
    windows = ((0, 0), (4096, 1 << 48))
    o_scan = [oracle.closure_scan(ranges, views, win_lo=w[0], win_hi=w[1], oob_cap=60) for w in windows]
    for shape in SHAPES:
        print(f"[gpu-case] hash shapes: {n_ranges} ranges, unit {unit}, {shape}", flush=True)
        sys.stdout.flush()
        ctx = kc.Context(0)
        for op_ in (kc.OP_SNAPSHOT, kc.OP_PAGE_HASH):
            ctx.set_tuning(op_, **shape)
        rs = kc.RangeSet(ctx, ranges, unit=unit)
        for w, expect in [(None, None)] + list(zip(windows, o_scan)):
            scan = kc.ScanOut("cuda", 60, *w) if w else None
            s = kc.snapshot(ctx, rs, seed=3, scan=scan)
            assert np.array_equal(u64(s["hash"])[: rs.n_pages], oh) and np.array_equal(u64(s["zero_bm"])[: rs.n_words], oz)
            assert int(u64(s["n_kept"])[0]) == onk and np.array_equal(u64(s["page_va"])[:onk], ova)
            assert np.array_equal(s["packed"][: onk * unit].cpu().numpy(), op)
            assert scan is None or scan.result() == expect
            for p in (None, torch.from_numpy(prior.view(np.int64)).cuda()):
                scan = kc.ScanOut("cuda", 60, *w) if w else None
                h, z, c = kc.page_hash(ctx, rs, seed=3, prior=p, scan=scan)
                assert np.array_equal(u64(h)[: rs.n_pages], oh) and np.array_equal(u64(z)[: rs.n_words], oz)
                assert p is None or np.array_equal(u64(c)[: rs.n_words], oc)
                assert scan is None or scan.result() == expect
        rs.close()
        ctx.close()
