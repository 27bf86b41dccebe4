"""The closure scan and the pointer graph search a wave's pointer-like words 64
at a time: word counts around 64 per tile, every word a pointer, one target
and many, tiles of one to sixteen pages and partial last pages, against the
oracle (whole numbers: no tolerance).

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


@pytest.mark.parametrize("per_tile,targets", [(1, 1), (63, 3), (64, 60), (65, 1), (129, 60), (4096, 2), (8192, 1),
                                              (8192, 60)])
def test_pointer_counts_per_tile(kc, per_tile, targets):
    say(f"closure scan and pointer graph: {per_tile} pointer words per 16-page tile, {targets} targets")
    rng = np.random.default_rng(per_tile * 100 + targets)
    sizes = np.concatenate([np.arange(1, 18), [16, 32, 33, 48], rng.integers(1, 40, size=40)]) * PAGE
    sizes[5::4] -= rng.integers(1, PAGE, size=len(sizes[5::4]))
    lay = W.make_layout(rng, sizes, gap_pages=(1, 3))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    content = np.zeros(lay.arena_bytes, dtype=np.uint8)
    words = content[:lay.arena_bytes // 8 * 8].view(np.uint64)
    words[:] = rng.integers(1, 1 << 20, size=len(words), dtype=np.uint64)   # never pointer-like
    for a, o in enumerate(lay.offsets):
        for t in range(0, int(sizes[a]), 16 * PAGE):
            n = min(16 * PAGE, int(sizes[a]) - t) // 8
            if n == 0:
                continue
            at = rng.choice(n, size=min(per_tile, n), replace=False) + (int(o) + t) // 8
            to = rng.integers(0, targets, size=len(at))
            words[at] = np.array([ranges[i][0] for i in to], dtype=np.uint64) + rng.integers(0, PAGE - 8, size=len(at)).astype(np.uint64)
            if len(at) > 1:  # one past a range's end: out of range
                words[at[0]] = np.uint64(ranges[a][0] + ranges[a][1])
    arena.buf.copy_(torch.from_numpy(content))
    views = W.host_views(lay, content)
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    for _ in range(2):
        scan = kc.ScanOut("cuda", oob_cap=40)
        kc.closure_scan(ctx, rs, scan)
        edge = kc.pointer_graph(ctx, rs)
        torch.cuda.synchronize()
        assert scan.result() == oracle.closure_scan(ranges, views, oob_cap=40)
        assert np.array_equal(edge.cpu().numpy().view(np.uint64), oracle.pointer_graph(ranges, views))
    rs.close()
    ctx.close()
