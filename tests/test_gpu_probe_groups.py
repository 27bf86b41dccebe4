"""The zero probe of a full snapshot: groups of 64 pages or 16 larger units, one
to sixteen waves per group, units whose only non-zero byte sits at the ends of
the probe's first 16 bytes, of a 1 KiB load, of a 4 KiB block and of the unit,
partial last units, ranges of one unit (64 tiles in a bitmap word).  The bitmap
against the bytes, the whole snapshot of the smaller sets against the oracle
(whole numbers and bytes: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PAGE = 4096
MiB = 1 << 20


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


def u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


# n_ranges, most units per range, unit
@pytest.mark.parametrize("n_ranges,most,unit", [(1, 1, PAGE), (70, 1, PAGE), (130, 3, PAGE), (40, 200, PAGE),
                                                (3, 180000, PAGE), (2, 300000, PAGE), (60, 20, 2 * PAGE),
                                                (30, 9, 64 << 10), (9, 5, 2 * MiB), (2, 12000, 2 * PAGE)])
def test_zero_bitmap_of_groups(kc, n_ranges, most, unit):
    print(f"[gpu-case] zero probe: {n_ranges} ranges of up to {most} units of {unit}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n_ranges * 1000003 + most + unit)
    units = rng.integers(max(1, most // 2), most + 1, size=n_ranges)
    sizes = units * unit - np.where(rng.random(n_ranges) < 0.5, rng.choice([1, 8, 17, 1000, 4081, 4095], size=n_ranges), 0)
    lay = W.make_layout(rng, sizes, gap_pages=(0, 2))
    arena = W.Arena(lay, "cuda")
    ranges = lay.ranges(arena.va_base)
    host = np.zeros(lay.arena_bytes, dtype=np.uint8)
    views = W.host_views(lay, host)
    places = [0, 15, 16, 1023, 1024, 4095, 4096, 16384, unit - 17, unit - 1]
    expect = []
    for v, size in zip(views, sizes):
        n = -(-int(size) // unit)
        kinds = rng.integers(0, 3, size=n)      # zero, one byte set, set from the start
        if n > 1000:
            kinds[rng.random(n) < 0.7] = 2
        at = np.arange(n) * unit + np.array(places)[rng.integers(0, len(places), size=n)] % unit
        one = (kinds == 1) & (at < size)
        v[at[one]] = 1
        v[np.flatnonzero(kinds == 2) * unit] = 7
        expect.append(~(one | (kinds == 2)))
    expect = np.concatenate(expect)
    arena.buf.copy_(torch.from_numpy(host))
    ctx = kc.Context(0)
    rs = kc.RangeSet(ctx, ranges, unit=unit)
    assert rs.n_pages == len(expect)
    scan = kc.ScanOut("cuda", oob_cap=8)
    for _ in range(2):  # the second call finds the first one's bitmap and counts
        s = kc.snapshot(ctx, rs, seed=5, scan=scan)
    got = u64(s["zero_bm"])[: rs.n_words]
    bits = np.unpackbits(got.view(np.uint8), bitorder="little").astype(bool)
    assert np.array_equal(bits[: len(expect)], expect)
    assert not bits[len(expect):].any()
    kept = int((~expect).sum())
    assert int(u64(s["n_kept"])[0]) == kept
    assert scan.result() == oracle.closure_scan(ranges, views, oob_cap=8)
    if sizes.sum() < 64 * MiB:
        oh, oz, _ = oracle.page_hash(ranges, views, seed=5, unit=unit)
        op, ova, onk = oracle.compact(ranges, views, oz, unit=unit)
        assert np.array_equal(got, oz) and onk == kept
        assert np.array_equal(u64(s["hash"])[: rs.n_pages], oh)
        assert np.array_equal(u64(s["page_va"])[:onk], ova)
        assert np.array_equal(s["packed"][: onk * unit].cpu().numpy(), op)
    rs.close()
    ctx.close()
