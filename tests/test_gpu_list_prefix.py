"""The list of out-of-range words on both sides of its two limits: up to 196,608
scan tiles the blocks sum up the counts before theirs, above that a prefix per
tile is made, and above 262,144 there are two blocks per compute unit.  Many entries:
several in a tile, in neighbouring tiles, in blocks apart, in the first and the
last, with capacities below, at and above their number, against the oracle
(whole numbers and order: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE = 4096


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


@pytest.mark.parametrize("n", [3000, 196_608, 196_609, 262_144, 262_700])
def test_lists_of_many_tiles(kc, n):
    print(f"[gpu-case] out-of-range list: {n} ranges of one tile", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n)
    sizes = np.full(n, 64)
    sizes[::997] = PAGE
    lay = W.make_layout(rng, sizes, gap_pages=(0, 1))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = np.zeros(-(-lay.arena_bytes // 8) * 8, dtype=np.uint8)
    words = host.view(np.uint64)
    first = np.asarray(lay.offsets) // 8
    past = np.uint64(ranges[0][0] - 64)  # below every range, inside the default window
    tiles = np.unique(np.concatenate([[0, 1, 2, n - 1, n - 2], rng.integers(0, n, size=400), np.arange(n // 2, n // 2 + 70),
                                      np.arange(0, n, 997)[:60], [min(n - 1, k * 1024 + d) for k in range(1, 257) for d in (-1, 0)]]))
    for t in tiles:
        some = rng.choice(int(sizes[t]) // 8, size=int(rng.integers(1, 9)), replace=False)
        words[first[t] + some] = past - rng.integers(0, 1000, size=len(some)).astype(np.uint64)
    inside = rng.integers(0, n, size=200)
    words[first[inside] + rng.integers(0, 8, size=200)] = np.uint64(ranges[n // 3][0])
    arena.buf.copy_(torch.from_numpy(host[:lay.arena_bytes]))
    views = W.host_views(lay, host[:lay.arena_bytes])
    total = oracle.closure_scan(ranges, views, oob_cap=1)[0]["n_oob"]
    assert total > 500
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    for cap in (1, 100, total - 1, total, total + 50):
        expect = oracle.closure_scan(ranges, views, oob_cap=cap)
        scan = kc.ScanOut("cuda", oob_cap=cap)
        kc.closure_scan(ctx, rs, scan)
        assert scan.result() == expect, cap
        scan = kc.ScanOut("cuda", oob_cap=cap)
        kc.page_hash(ctx, rs, scan=scan)
        assert scan.result() == expect, cap
    rs.close()
    ctx.close()
