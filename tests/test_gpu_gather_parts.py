"""The gather of a delta, 64 KiB of a tile per wave: units from 4 KiB to 2 MiB,
tiles of 8 and 16 units, partial last units that end before, at and inside a
4 KiB block, no, some and all units kept, capacities below the kept count,
against the oracle (whole numbers and bytes: no tolerance).

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


@pytest.mark.parametrize("unit,n_ranges,most", [(PAGE, 50, 40), (2 * PAGE, 30, 40), (2 * PAGE, 2500, 4), (32 * KiB, 20, 20),
                                                (64 * KiB, 20, 20), (128 * KiB, 8, 18), (2 * MiB, 3, 10)])
def test_gather_parts(kc, unit, n_ranges, most):
    print(f"[gpu-case] gather: {n_ranges} ranges of up to {most} units of {unit}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(unit + n_ranges + most)
    sizes = rng.integers(1, most + 1, size=n_ranges) * unit
    cut = rng.choice([1, 17, 4095, 4096, unit - 4096, unit - 4095, unit - 1], size=n_ranges)
    sizes = sizes - np.where(rng.random(n_ranges) < 0.5, np.minimum(cut, unit - 1), 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(1, 256, size=lay.arena_bytes, dtype=np.uint8)
    views = W.host_views(lay, host)
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    prior, _, _ = kc.page_hash(ctx, rs)
    for share in (0.0, 0.3, 1.0):
        for v in views:
            for u in np.flatnonzero(rng.random(-(-len(v) // unit)) < share):
                v[min(len(v) - 1, u * unit + int(rng.integers(0, unit)))] ^= 0x55
        arena.buf.copy_(torch.from_numpy(host))
        h, z, c = kc.page_hash(ctx, rs, prior=prior)
        oh, oz, oc = oracle.page_hash(ranges, views, prior=u64(prior)[:rs.n_pages], unit=unit)
        assert np.array_equal(u64(c)[:rs.n_words], oc)
        kept = int(np.bitwise_count(oc & ~oz).sum())
        for cap in sorted({rs.n_pages, max(1, kept // 2)}):
            s = kc.snapshot(ctx, rs, prior=prior, cap_pages=cap)
            op, ova, onk = oracle.compact(ranges, views, oz, oc, cap_pages=cap, unit=unit)
            k = min(onk, cap)
            assert int(u64(s["n_kept"])[0]) == onk
            assert np.array_equal(u64(s["page_va"])[:k], ova)
            assert np.array_equal(s["packed"][:k * unit].cpu().numpy(), op)
    rs.close()
    ctx.close()


@pytest.mark.parametrize("unit,n_ranges,most", [(16 * KiB, 16500, 2 * PAGE), (64 * KiB, 4200, 20 * PAGE), (2 * MiB, 270, 5 * PAGE)])
def test_gather_long_parts(kc, unit, n_ranges, most):
    """So many tiles of larger units that a wave takes 256 KiB of one: mostly
    ranges under a unit, some of several."""
    print(f"[gpu-case] gather: {n_ranges} ranges, units of {unit}, long parts", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(unit + n_ranges)
    sizes = rng.integers(1, most + 1, size=n_ranges)
    long_ones = rng.choice(n_ranges, size=6, replace=False)
    sizes[long_ones] = rng.integers(1, 4, size=6) * unit + rng.choice([0, 1, 4096, unit - 4095], size=6)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = rng.integers(1, 256, size=lay.arena_bytes, dtype=np.uint8)
    views = W.host_views(lay, host)
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    zb = np.zeros(rs.n_words, dtype=np.uint64)
    for share in (0.0, 0.02, 0.7, 1.0):
        keep = rng.random(rs.n_pages) < share
        zb[:] = np.packbits(~np.pad(keep, (0, rs.n_words * 64 - rs.n_pages)), bitorder="little").view(np.uint64)
        zb[-1] &= np.uint64((1 << (rs.n_pages - 64 * (rs.n_words - 1))) - 1)
        for grid in (0, 1):
            ctx.set_tuning(kc.OP_COMPACT, grid_per_cu=grid)
            packed, va, nk = kc.compact(ctx, rs, torch.from_numpy(zb.view(np.int64)).cuda(), cap_pages=max(1, int(keep.sum())))
            op, ova, onk = oracle.compact(ranges, views, zb, cap_pages=max(1, int(keep.sum())), unit=unit)
            assert int(u64(nk)[0]) == onk == int(keep.sum())
            assert np.array_equal(u64(va)[:onk], ova[:onk])
            assert np.array_equal(packed[:onk * unit].cpu().numpy(), op[:onk * unit])
    rs.close()
    ctx.close()
