"""Launch shapes of the compare at the lines between them: as many pairs as
compute units and one more, pairs of 64 KiB and one element more, batches of a
little under and over two tiles of each size per compute unit.  Every report
equals the oracle's (integers and exact fp64 maxima: no tolerance).

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
KiB = 1 << 10


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


# pairs (0: one per CU, -1: one more) and bytes of a pair (negative: that many times the number of CUs)
@pytest.mark.parametrize("n_pairs,size", [(0, 64 * KiB), (0, 64 * KiB + 2), (-1, 300), (3, -8 * KiB), (3, -11 * KiB),
                                          (5, -12 * KiB), (2, -70 * KiB), (1, -64 * KiB)])
def test_compare_launch_shapes(kc, n_pairs, size):
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n_pairs < 1:
        n_pairs = cu - n_pairs
    if size < 0:
        size = -size * cu
    print(f"[gpu-case] compare shapes: {n_pairs} pairs of {size} bytes", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n_pairs + size)
    dt = next(d for d in W.TORCH_DTYPE if W.TORCH_DTYPE[d] == torch.bfloat16)
    n = size // 2
    gold = (torch.randn(n, generator=torch.Generator().manual_seed(size % 1000))).to(torch.bfloat16)
    raw = gold.view(torch.int16).numpy()
    gold_d = gold.view(torch.uint8).cuda()
    host, pairs = [], []
    for i in range(n_pairs):
        cand = raw.copy()
        at = rng.integers(0, n, size=1 + (n // 997 if i % 3 == 0 else 0))
        cand[at] ^= rng.integers(1, 8, size=len(at)).astype(np.int16)
        if i < 8 or i >= n_pairs - 2:   # the oracle looks at the first ones and the last
            host.append((i, cand.view(np.uint8)))
        pairs.append((torch.from_numpy(cand.view(np.uint8)).cuda(), gold_d, dt, i % 4, 1e-3, 1e-2))
    ctx = kc.Context(0)
    want = {i: oracle.compare(c, raw.view(np.uint8), dt, i % 4, 1e-3, 1e-2) for i, c in host}
    ps = kc.PairSet(ctx, pairs)
    got = [kc.decode_cmp(kc.compare(ctx, pairs), n_pairs), kc.decode_cmp(kc.compare_pairset(ctx, ps), n_pairs)]
    if n_pairs <= kc.NOALLOC_MAX_PAIRS:
        res = torch.zeros(n_pairs * kc.RESULT_BYTES, dtype=torch.uint8, device="cuda")
        got.append(kc.decode_cmp(kc.compare_noalloc(ctx, pairs, res), n_pairs))
    for g in got:
        assert g == got[0]
        assert {i: g[i] for i in want} == want
    ps.close()
    ctx.close()
