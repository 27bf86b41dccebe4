"""The hashing pass at each number of units per wave (4, 8 and 16, chosen by
the number of tiles) and of waves per workgroup: range sets of few, some and
many tiles, ranges that end at and around parts of a tile, partial last pages of
under and over a stripe, pages and larger units, with and without the scan and
the prior table, against the oracle (whole numbers and bytes: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE = 4096


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n_ranges,unit", [(3, PAGE), (60, PAGE), (300, PAGE), (1300, PAGE), (900, 2 * PAGE), (2400, 2 * PAGE),
                                           (40, 16 * PAGE)])
def test_rows_parts_and_partial_units(kc, n_ranges, unit):
    rng = np.random.default_rng(n_ranges + unit)
    units = rng.choice([1, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17], size=n_ranges)
    sizes = units * unit
    cut = rng.choice([0, 1, 8, 17, 31, 32, 33, 1000, 1024, 2048, 4064, 4095], size=n_ranges)  # bytes off the end
    sizes = sizes - np.where(rng.random(n_ranges) < 0.6, cut, 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(0, 256, size=lay.arena_bytes, dtype=np.uint8)
    words = host[: lay.arena_bytes // 8 * 8].view(np.uint64)
    at = rng.choice(len(words), size=max(4, len(words) // 300), replace=False)
    to = rng.integers(0, n_ranges, size=len(at))
    words[at] = np.array([ranges[i][0] + ranges[i][1] * (j % 3 == 0) for j, i in enumerate(to)], dtype=np.uint64)
    zero = rng.random(lay.arena_bytes // unit + 1) < 0.25
    for i in np.flatnonzero(zero):
        host[i * unit:(i + 1) * unit] = 0
    arena.buf.copy_(torch.from_numpy(host))
    views = W.host_views(lay, host)
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    oh, oz, _ = oracle.page_hash(ranges, views, seed=3, unit=unit)
    op, ova, onk = oracle.compact(ranges, views, oz, unit=unit)
    o_scan = oracle.closure_scan(ranges, views, oob_cap=50)
    prior = oh.copy()
    prior[::5] ^= np.uint64(1)
    for scanned in (False, True):
        say(f"hash rows: {n_ranges} ranges, unit {unit}, scan {scanned}")
        scan = kc.ScanOut("cuda", oob_cap=50) if scanned else None
        s = kc.snapshot(ctx, rs, seed=3, scan=scan)
        assert np.array_equal(u64(s["hash"])[: rs.n_pages], oh)
        assert np.array_equal(u64(s["zero_bm"])[: rs.n_words], oz)
        assert int(u64(s["n_kept"])[0]) == onk
        assert np.array_equal(u64(s["page_va"])[:onk], ova)
        assert np.array_equal(s["packed"][: onk * unit].cpu().numpy(), op)
        assert scan is None or scan.result() == o_scan
        scan = kc.ScanOut("cuda", oob_cap=50) if scanned else None
        h, z, c = kc.page_hash(ctx, rs, seed=3, prior=torch.from_numpy(prior.view(np.int64)).cuda(), scan=scan)
        assert np.array_equal(u64(h)[: rs.n_pages], oh)
        assert np.array_equal(u64(z)[: rs.n_words], oz)
        assert np.array_equal(np.flatnonzero(np.unpackbits(u64(c).view(np.uint8), bitorder="little")[: rs.n_pages]),
                              np.arange(rs.n_pages)[::5])
        assert scan is None or scan.result() == o_scan
    rs.close()
    ctx.close()
