"""Candidate materialisation where its pieces (8 KiB), short last vectors and
block sizes end: lengths around whole pieces, blocks from the shortest that the
piece-wise kernel takes to longer than a buffer (and one below it), against a
copy moved by the seeded generator on the CPU.  Bits are equal: no tolerance.

Every case prints its name before touching the GPU."""
import sys

import numpy as np
import pytest
import torch

from paper_2605_03208_amd import workloads as W

pytestmark = pytest.mark.gpu
PIECE = 8192


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def kc():
    from paper_2605_03208_amd import kc as K
    K.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return K


@pytest.mark.parametrize("dt", [W.DT_F64, W.DT_F32, W.DT_F16, W.DT_FP8, W.DT_I8])
def test_pieces_short_vectors_and_blocks(kc, dt):
    w = W.ELEM_SIZE[dt]
    rng = np.random.default_rng(40 + dt)
    per = PIECE // w
    lens = np.array([per - 1, per, per + 1, 2 * per + 16 // w + 1, 3 * per - 16 // w + 1, 5 * per + 7, 1, 20 * per + 3])
    raw = torch.from_numpy(rng.integers(0, 256, size=int(lens.sum()) * w, dtype=np.uint8)).view(W.TORCH_DTYPE[dt])
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]])
    golds = [raw[a: a + n].to("cuda") for a, n in zip(starts.tolist(), lens.tolist())]
    step = 16 // w
    room = -(-lens // step) * step + step        # a gap after every buffer
    offs = np.concatenate([[0], np.cumsum(room)[:-1]]).astype(np.int64)
    bits = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[w]
    ctx = kc.Context(0)
    for block in (256 // w - 1, 256 // w, 256 // w + 1, 997, per, 10000, 30 * per):
        say(f"kc_materialize pieces: dtype {dt}, block {block}")
        seeds = rng.integers(0, 2**31, size=len(lens))
        arena = torch.full((int(room.sum()) * w,), 0x5A, dtype=torch.uint8, device="cuda").view(raw.dtype)
        want = arena.cpu().clone()
        for a, n, o in zip(starts.tolist(), lens.tolist(), offs.tolist()):
            want[o: o + n] = raw[a: a + n]
        W.perturb_many(want, dt, offs, lens, seeds, 1.0 / block, 16)
        kc.materialize(ctx, arena, [g.data_ptr() for g in golds], offs, lens, seeds, block, 16)
        torch.cuda.synchronize()
        assert torch.equal(arena.cpu().view(bits), want.view(bits)), block
    ctx.close()


@pytest.mark.parametrize("dt", [W.DT_F64, W.DT_BF16, W.DT_FP8])
@pytest.mark.parametrize("mib", [False, True])
def test_lines_between_the_forms(kc, dt, mib):
    """Blocks around 512 bytes and 1 KiB, buffers of under and over 1 MiB on
    average: the shorter blocks take the form by vectors."""
    w = W.ELEM_SIZE[dt]
    rng = np.random.default_rng(400 + dt + mib)
    lens = rng.integers(900_000, 1_300_000, size=3) // w + (200_000 // w if mib else -300_000 // w)
    lens = np.concatenate([lens, [1, 5000 // w]] if not mib else [lens])
    raw = torch.from_numpy(rng.integers(0, 256, size=int(lens.sum()) * w, dtype=np.uint8)).view(W.TORCH_DTYPE[dt])
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]])
    golds = [raw[a: a + n].to("cuda") for a, n in zip(starts.tolist(), lens.tolist())]
    room = -(-lens // (16 // w)) * (16 // w) + 16 // w
    offs = np.concatenate([[0], np.cumsum(room)[:-1]]).astype(np.int64)
    bits = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[w]
    ctx = kc.Context(0)
    for block in (512 // w - 1, 512 // w, 1024 // w - 1, 1024 // w):
        say(f"kc_materialize forms: dtype {dt}, block {block}, buffers of 1 MiB {mib}")
        seeds = rng.integers(0, 2**31, size=len(lens))
        arena = torch.full((int(room.sum()) * w,), 0x5A, dtype=torch.uint8, device="cuda").view(raw.dtype)
        want = arena.cpu().clone()
        for a, n, o in zip(starts.tolist(), lens.tolist(), offs.tolist()):
            want[o: o + n] = raw[a: a + n]
        W.perturb_many(want, dt, offs, lens, seeds, 1.0 / block, 16)
        kc.materialize(ctx, arena, [g.data_ptr() for g in golds], offs, lens, seeds, block, 16)
        torch.cuda.synchronize()
        assert torch.equal(arena.cpu().view(bits), want.view(bits)), block
    ctx.close()


def test_short_blocks_time(kc):
    """Short blocks do not make a call much longer than long ones: of pieces whose moves are applied one by one they
    do."""
    n, el = 2000, 20000
    raw = torch.randint(0, 100, (n * el,), dtype=torch.uint8, device="cuda")
    arena = torch.zeros_like(raw).view(torch.float8_e4m3fn)
    offs = np.arange(n) * el
    src = np.uint64(raw.data_ptr()) + offs.astype(np.uint64)
    ctx = kc.Context(0)
    us = {}
    for block in (250, 300, 400, 4096):
        say(f"kc_materialize forms: time, block {block}")
        call = lambda: kc.materialize(ctx, arena, src, offs, np.full(n, el), np.arange(n), block, 16)
        call()
        ms = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        us[block] = min(ms) * 1e3
    say(f"kc_materialize forms: {us}")
    assert max(us[300], us[400]) < 1.25 * us[250]
    ctx.close()
