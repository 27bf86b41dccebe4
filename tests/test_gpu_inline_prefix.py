"""Prefixes that the consuming kernels count themselves: packed slots of snapshots
around 512 bitmap words, and lists of out-of-range words over one to a few
thousand tiles with caps around the number of entries, dense and sparse, against
the oracle (whole numbers and bytes: no tolerance).

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


def state(kc, rng, sizes):
    lay = W.make_layout(rng, np.asarray(sizes), gap_pages=(1, 3))
    arena = W.Arena(lay, "cuda")
    host = np.zeros(lay.arena_bytes, dtype=np.uint8)
    return lay, arena, lay.ranges(arena.va_base), host, W.host_views(lay, host)


@pytest.mark.parametrize("n_pages,cap", [(1, None), (63, None), (64, 20), (65, None), (511 * 64 + 63, None),
                                         (512 * 64, 10000), (512 * 64 + 1, None), (513 * 64, 10000)])
def test_slots_around_the_word_limit(kc, n_pages, cap):
    say(f"slots of {n_pages} pages, capacity {cap}")
    rng = np.random.default_rng(n_pages)
    parts = sorted(rng.choice(np.arange(1, n_pages), size=min(9, n_pages - 1), replace=False)) if n_pages > 1 else []
    sizes = np.diff([0, *parts, n_pages]) * PAGE
    lay, arena, ranges, host, views = state(kc, rng, sizes)
    for v in views:
        kinds = rng.integers(0, 3, size=len(v) // PAGE)
        v[np.flatnonzero(kinds > 0) * PAGE + rng.integers(0, PAGE)] = 1 + rng.integers(0, 255)
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    s = kc.snapshot(ctx, rs, seed=9, cap_pages=cap)
    oh, oz, _ = oracle.page_hash(ranges, views, seed=9)
    op, ova, onk = oracle.compact(ranges, views, oz, cap_pages=cap)
    k = min(onk, n_pages if cap is None else cap)
    assert int(u64(s["n_kept"])[0]) == onk
    assert np.array_equal(u64(s["hash"])[: rs.n_pages], oh)
    assert np.array_equal(u64(s["page_va"])[:k], ova)
    assert np.array_equal(s["packed"][: k * PAGE].cpu().numpy(), op)
    rs.close()
    ctx.close()


# tiles: one per range; entries: per tile with some; every: one such tile in so many
@pytest.mark.parametrize("n_tiles,entries,every", [(1, 3, 1), (4, 1, 2), (255, 2, 7), (256, 1, 1), (257, 300, 1),
                                                   (1030, 5, 1), (3000, 1, 97), (3000, 40, 3)])
def test_out_of_range_lists(kc, n_tiles, entries, every):
    rng = np.random.default_rng(n_tiles * 7 + entries)
    sizes = rng.integers(1, 17, size=n_tiles) * PAGE - rng.choice([0, 8, 20, 4000], size=n_tiles)
    lay, arena, ranges, host, views = state(kc, rng, sizes)
    total = 0
    for i, v in enumerate(views):
        words = v[: len(v) // 8 * 8].view(np.uint64)
        words[:: max(1, len(words) // 3)] = ranges[rng.integers(0, n_tiles)][0]     # in range
        if i % every == every - 1:
            n = min(entries, len(words))
            words[rng.choice(len(words), size=n, replace=False)] = ranges[i][0] + ranges[i][1]  # just past the end
            total += n
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    for cap in sorted({0, 1, max(1, total // 2), max(1, total - 1), total, total + 1, 2 * total + 5}):
        say(f"list of {total} out-of-range words over {n_tiles} tiles, capacity {cap}")
        expect = oracle.closure_scan(ranges, views, oob_cap=cap)
        scan = kc.ScanOut("cuda", oob_cap=cap)
        kc.snapshot(ctx, rs, scan=scan)
        assert scan.result() == expect
        scan = kc.ScanOut("cuda", oob_cap=cap)
        kc.closure_scan(ctx, rs, scan)
        assert scan.result() == expect
    rs.close()
    ctx.close()
