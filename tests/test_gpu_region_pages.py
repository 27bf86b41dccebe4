"""The region diff of pages at the lines of its launch: groups of four tiles
around one per compute unit and around one to four waves per workgroup, runs of
several groups per wave, ranges that end inside a wave's run, a workgroup's and
between workgroups, against the oracle (whole numbers: no tolerance).

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


@pytest.mark.parametrize("n_ranges,most", [(1, 1), (3, 1), (5, 1), (1021, 1), (1025, 2), (2049, 1), (4099, 1), (9001, 1), (3, 3000),
                                           (700, 60)])
def test_page_groups(kc, n_ranges, most):
    print(f"[gpu-case] region diff: {n_ranges} ranges of up to {most} pages", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n_ranges * 7 + most)
    sizes = rng.integers(1, most + 1, size=n_ranges) * PAGE
    sizes = sizes - np.where(rng.random(n_ranges) < 0.3, rng.integers(1, PAGE, size=n_ranges), 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(1, 256, size=lay.arena_bytes, dtype=np.uint8)
    views = W.host_views(lay, host)
    for v in views:
        if rng.random() < 0.2:
            v[:min(len(v), 5 * PAGE)] = 0
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges)
    gold = kc.snapshot(ctx, rs, seed=1)
    u64 = lambda t: t.detach().cpu().numpy().view(np.uint64)
    onk = int(u64(gold["n_kept"])[0])
    zb, pk, va = u64(gold["zero_bm"])[:rs.n_words].copy(), gold["packed"][:onk * PAGE].cpu().numpy(), u64(gold["page_va"])[:onk].copy()
    for share in (0.01, 0.5):
        for v in views:
            for g in np.flatnonzero(rng.random(-(-len(v) // PAGE)) < share):
                end = min(len(v), (g + 1) * PAGE)
                v[min(end - 1, g * PAGE + int(rng.choice([0, 15, 16, 1023, 1024, 4095])))] ^= 0x41
                if rng.random() < 0.3:
                    v[g * PAGE:end] += 1
        arena.buf.copy_(torch.from_numpy(host))
        for grid in (0, 1, 20):
            ctx.set_tuning(kc.OP_REGION_DIFF, grid_per_cu=grid)
            for cap in (onk, onk // 2):
                out = kc.region_diff(ctx, rs, gold, seed=1, cap_pages=cap)
                assert kc.decode_region_diff(out["res"], n_ranges) == oracle.region_diff(
                    ranges, views, zb, pk[:cap * PAGE], va[:cap], onk, cap_pages=cap)
    rs.close()
    ctx.close()
