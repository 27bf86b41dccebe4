"""How the tiles of a compare are shared out to workgroups: evenly, in runs of a
fixed length, and in runs that shrink towards the end of a long list of pairs.
Every report equals the oracle's on the lines between these (whole numbers and
exact fp64 maxima: no tolerance), and one wholly different pair among equal ones
does not keep the chip waiting, wherever it stands.

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
TILE = 4096
RUN = (512 << 10) // TILE      # tiles of a whole run at this tile size
TAPER = (RUN - 1) * 512        # tiles of the shrinking runs


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


@pytest.mark.parametrize("n_pairs,tiles", [(16, 2 * TAPER - 1), (16, 2 * TAPER), (40, 2 * TAPER + RUN + 1), (15, 2 * TAPER + 3)])
def test_runs_and_their_shrinking(kc, n_pairs, tiles):
    say(f"compare runs: {n_pairs} pairs, {tiles} tiles of {TILE} bytes")
    rng = np.random.default_rng(n_pairs + tiles)
    cuts = np.sort(rng.choice(np.arange(1, tiles), size=n_pairs - 1, replace=False))
    count = np.diff(np.concatenate([[0], cuts, [tiles]]))
    gold = torch.randint(0, 120, (tiles * TILE,), dtype=torch.uint8, device="cuda")
    cand = gold.clone()
    first = np.concatenate([[0], np.cumsum(count)]) * TILE
    last = int(first[-1])
    for a, b in ((0, 3 * TILE), (last - 40 * TILE, last), (last // 2, last // 2 + TILE)):  # wholly different stretches
        cand[a:b] ^= 5
    for at in np.concatenate([rng.integers(0, last, size=400), first[1:-1], first[1:] - 1]):
        cand[int(at)] ^= 2
    host_c, host_g = cand.cpu().numpy(), gold.cpu().numpy()
    pairs, expect = [], []
    for i in range(n_pairs):
        dt = (W.DT_F32, W.DT_BF16, W.DT_FP8, W.DT_I16)[i % 4]
        a, b = int(first[i]), int(first[i + 1]) - int(rng.integers(0, 3)) * 8
        pairs.append((cand[a:b], gold[a:b], dt, 2, 1e-3, 1e-2))
        expect.append(oracle.compare(host_c[a:b], host_g[a:b], dt, 2, 1e-3, 1e-2))
    ctx = kc.Context(0)
    for grid in (1, 0):
        ctx.set_tuning(kc.OP_COMPARE, grid_per_cu=grid, tile_bytes=TILE)
        assert kc.decode_cmp(kc.compare(ctx, pairs), n_pairs) == expect, grid
        res = torch.zeros(n_pairs * kc.RESULT_BYTES, dtype=torch.uint8, device="cuda")
        assert kc.decode_cmp(kc.compare_noalloc(ctx, pairs, res), n_pairs) == expect, grid
    ctx.set_tuning(kc.OP_COMPARE, grid_per_cu=1, tile_bytes=TILE, per_item=1)
    assert kc.decode_cmp(kc.compare(ctx, pairs), n_pairs) == expect
    ctx.close()


@pytest.mark.parametrize("shape", [dict(), dict(grid_per_cu=2, tile_bytes=131072)])
def test_one_wrong_pair_time(kc, shape):
    """200 pairs of 10 MiB, one of them all off: the call takes about as long as with none."""
    n, size = 200, 10 << 20
    gold = torch.randint(0, 120, (n * size,), dtype=torch.uint8, device="cuda")
    cand = gold.clone()
    ctx = kc.Context(0)
    ctx.set_tuning(kc.OP_COMPARE, **shape)
    ps = kc.PairSet(ctx, [(cand[i * size:(i + 1) * size], gold[i * size:(i + 1) * size], W.DT_FP8, 2, 1e-3, 1e-2)
                          for i in range(n)])
    res = kc.compare_pairset(ctx, ps)
    us = {}
    for wrong in (None, 0, n // 2, n - 1):
        say(f"compare runs: time, shape {shape}, pair {wrong} all off")
        if wrong is not None:
            cand[wrong * size:(wrong + 1) * size] ^= 1
        ms = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            kc.compare_pairset(ctx, ps, res)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        us[wrong] = min(ms[1:]) * 1e3
        if wrong is not None:
            cand[wrong * size:(wrong + 1) * size] ^= 1
    say(f"compare runs: {us}")
    for wrong in (0, n // 2, n - 1):
        assert us[wrong] < 1.4 * us[None], us
    ps.close()
    ctx.close()


def test_copies_of_the_accumulators(kc):
    """Lists on both sides of the lines from which pairs have several copies of
    their accumulators, through one context and one resident list each, in turn
    and again: every report equals that of its pair alone (a small list)."""
    rng = np.random.default_rng(3)
    total = (1 << 30) + (64 << 20)
    gold = torch.randint(0, 120, (total,), dtype=torch.uint8, device="cuda")
    cand = gold.clone()
    at = torch.from_numpy(rng.integers(0, total, size=200000)).cuda()
    cand[at] ^= 3
    lists = []
    for n, size in ((2, total), (1, 1 << 30), (40, total), (512, total), (513, total)):
        cuts = np.sort(rng.choice(np.arange(1, size // 4096), size=n - 1, replace=False)) * 4096
        first = np.concatenate([[0], cuts, [size]])
        lists.append([(cand[a:b], gold[a:b], (W.DT_FP8, W.DT_F32, W.DT_F16, W.DT_U8, W.DT_I64)[i % 5], 2, 1e-3, 1e-2)
                      for i, (a, b) in enumerate(zip(first[:-1].tolist(), first[1:].tolist()))])
    ctx = kc.Context(0)
    expect = []
    for pairs in lists:
        say(f"compare copies: {len(pairs)} pairs alone")
        expect.append([kc.decode_cmp(kc.compare(ctx, [p]), 1)[0] for p in pairs])
    resident = [kc.PairSet(ctx, pairs) for pairs in lists]
    for again in range(2):
        for pairs, ps, want in zip(lists, resident, expect):
            say(f"compare copies: {len(pairs)} pairs, time {again}")
            res = torch.zeros(len(pairs) * kc.RESULT_BYTES, dtype=torch.uint8, device="cuda")
            for got in (kc.compare(ctx, pairs), kc.compare_pairset(ctx, ps), kc.compare_noalloc(ctx, pairs, res)):
                assert kc.decode_cmp(got, len(pairs)) == want
    for ps in resident:
        ps.close()
    ctx.close()
