"""Bags of several lookups at the edges of what the kernels take at a time: the forward's 8 rows per request, the segment sums' 64
parked chunk sums, four to a load.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from helpers import GpuRun, assert_exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [8, 24, 40, 64, 72, 136, 256])
def test_forward_bag_lengths(oracle, D):
    rng = np.random.default_rng(D)
    lens = np.array([0, 1, 2, 7, 8, 9, 15, 16, 17, 24, 33])
    T, B = 3, 37  # (the last tile of 16 samples is partial)
    per_bag = rng.permuted(np.resize(lens, T * B))
    rows = np.array([1, 500, 70000])
    row_offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(per_bag)]).astype(np.int64)
    idx = np.concatenate([rng.integers(0, rows[t], per_bag[t * B:(t + 1) * B].sum()) for t in range(T)]).astype(np.int64)
    W = (rng.standard_normal((row_offsets[-1], D)) * 0.1).astype(np.float32)
    s = oracle.find_scale(W, row_offsets)
    expect, codes = oracle.embbag_fwd(W, None, row_offsets, s, B, idx, off)
    for want_codes in (False, True):
        run = GpuRun(row_offsets, D, W, B, len(idx), want_codes=want_codes)
        run.upload_batch(idx, off)
        run.set_scale(s)
        run.pack()
        for mode in (0, 1):
            out, got = run.fwd(mode)
            assert_exact(out.view(np.uint32), expect.view(np.uint32), f"out bits, mode {mode}")
            if want_codes:
                assert_exact(got, codes, f"codes, mode {mode}")
        assert run.status()[0] == 0


# rows of 2 .. 131 chunks of 32 lookups: one and two requests of 64 chunk sums, their remainders of four
@pytest.mark.parametrize("D", [8, 16, 40, 64, 72, 136, 256])
def test_segments_of_many_chunks(oracle, D):
    rng = np.random.default_rng(D)
    counts = np.array([33, 64, 65, 97, 129, 32 * 64, 32 * 64 + 1, 32 * 65 + 1, 32 * 68, 32 * 130 + 7, 1, 2])
    T, B, L = 1, 1600, int(-(-counts.sum() // 1600))
    rows = np.repeat(np.arange(len(counts)), counts)
    idx = rng.permutation(np.concatenate([rows, np.zeros(B * L - len(rows), np.int64)])).astype(np.int64)
    off = (np.arange(B + 1) * L).astype(np.int64)
    row_offsets = np.array([0, len(counts)], np.int64)
    g = (rng.standard_normal((B, T, D)) * 1e-4).astype(np.float32)
    run = GpuRun(row_offsets, D, np.zeros((len(counts), D), np.float32), B, len(idx))
    run.upload_batch(idx, off, g)
    got, o = run.bwd(), oracle.embbag_bwd(T, D, B, idx, off, g)
    U = got["U"]
    assert U == len(counts)
    assert_exact(got["values"][:U].view(np.uint32), o["values"][:U].view(np.uint32), "values bits")
    assert_exact(got["g_absmax"].view(np.uint32), o["g_absmax"].view(np.uint32), "absmax bits")
    assert run.status()[0] == 0


# Segments of 2 .. 5 chunks that are the whole batch: one full chunk and a last one, up to more than one load of four, in a workspace
# of exactly the size asked for.  What lies behind it is NaN and stays as it is.
@pytest.mark.parametrize("n", [33, 64, 65, 128, 129, 160])
@pytest.mark.parametrize("D", [40, 64, 72, 256])
def test_one_segment_in_a_workspace_of_the_size_asked_for(oracle, D, n):
    import torch

    row_offsets, off = np.array([0, 1], np.int64), np.arange(n + 1, dtype=np.int64)
    g = (np.random.default_rng(n).standard_normal((n, 1, D)) * 1e-4).astype(np.float32)
    run = GpuRun(row_offsets, D, np.zeros((1, D), np.float32), n, n)
    run.upload_batch(np.zeros(n, np.int64), off, g)
    size = run.bufs.workspace.numel()
    room = torch.full((size + 32768,), 0xFF, dtype=torch.uint8, device=run.dev)
    run.bufs.workspace = room[:size]
    got, o = run.bwd(), oracle.embbag_bwd(1, D, n, np.zeros(n, np.int64), off, g)
    assert got["U"] == 1
    assert_exact(got["values"][:1].view(np.uint32), o["values"][:1].view(np.uint32), "values bits")
    assert_exact(got["g_absmax"].view(np.uint32), o["g_absmax"].view(np.uint32), "absmax bits")
    assert bool((room[size:] == 0xFF).all())
    assert run.status()[0] == 0
