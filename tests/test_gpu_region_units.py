"""The region diff over units from 4 KiB to 2 MiB: one to sixteen waves per
group, differing bytes at the ends of 4 KiB blocks, of units and of partial last
units, units that were or become zero, runs of unchanged groups between changed
ones, slots beyond the capacity, against the oracle (whole numbers: no
tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE = 4096
KiB, MiB = 1 << 10, 1 << 20


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("unit,n_ranges,most", [(PAGE, 70, 40), (PAGE, 2, 9000), (16 * KiB, 40, 30), (32 * KiB, 9, 40),
                                                (64 * KiB, 300, 3), (64 * KiB, 2, 500), (256 * KiB, 5, 20), (2 * MiB, 4, 9)])
def test_region_diff_units(kc, unit, n_ranges, most):
    print(f"[gpu-case] region diff: {n_ranges} ranges of up to {most} units of {unit}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(unit + n_ranges * 31 + most)
    sizes = rng.integers(1, most + 1, size=n_ranges) * unit
    sizes = sizes - np.where(rng.random(n_ranges) < 0.5, rng.choice([1, 8, 17, 1000, 4081, 4095], size=n_ranges), 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(1, 256, size=lay.arena_bytes, dtype=np.uint8)
    views = W.host_views(lay, host)
    for v in views:
        for u in np.flatnonzero(rng.random(-(-len(v) // unit)) < 0.2):
            v[u * unit:(u + 1) * unit] = 0
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    gold = kc.snapshot(ctx, rs, seed=1)
    onk = int(u64(gold["n_kept"])[0])
    zb, pk, va = u64(gold["zero_bm"])[:rs.n_words].copy(), gold["packed"][:onk * unit].cpu().numpy(), u64(gold["page_va"])[:onk].copy()
    for share in (0.02, 0.6, 1.0):
        for v in views:
            for u in np.flatnonzero(rng.random(-(-len(v) // unit)) < share):
                end = min(len(v), (u + 1) * unit)
                at = u * unit + np.array([0, 15, 16, 4095, 4096, 16383, unit // 2, unit - 1])
                kind = rng.integers(0, 4)
                if kind == 0:
                    v[u * unit:end] = 0
                elif kind == 1:
                    v[u * unit:end] += 1
                else:
                    v[np.minimum(rng.choice(at, size=kind), end - 1)] ^= 0x41
        arena.buf.copy_(torch.from_numpy(host))
        for cap in (onk, onk // 2):
            out = kc.region_diff(ctx, rs, gold, seed=1, cap_pages=cap)
            got = kc.decode_region_diff(out["res"], n_ranges)
            assert got == oracle.region_diff(ranges, views, zb, pk[:cap * unit], va[:cap], onk, cap_pages=cap, unit=unit)
    rs.close()
    ctx.close()
