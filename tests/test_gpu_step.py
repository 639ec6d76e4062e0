"""dqrm_fwd_bwd_step against the calls that it stands for (forward, backward with maxima, INT8 codes, update), bit for bit in every
buffer and table."""
import numpy as np
import pytest

from helpers import GpuRun, assert_exact

pytestmark = pytest.mark.gpu

NAMES = ("out", "codes", "sorted_pos", "uniq_rows", "seg_offsets", "table_uniq_offsets", "num_unique", "values", "g_absmax", "gq", "g_scale")


def _batch(rng, rows, B, lens):
    per_table = [lens(len(rows), t, B) for t in range(len(rows))]
    off = np.concatenate([[0], np.cumsum(np.concatenate(per_table))]).astype(np.int64)
    idx = np.concatenate([rng.integers(0, max(r, 1), n.sum()) for r, n in zip(rows, per_table)]).astype(np.int64)
    return idx, off


def _runs(rows, D, B, idx, off, grad, mode, cap=None):
    """The same step twice from the same tables: in one call, and in its parts."""
    import torch
    import paper_2410_20046_amd as dq

    row_offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    W = (np.random.default_rng(5).standard_normal((row_offsets[-1], D)) * 0.1).astype(np.float32)
    results = []
    for one_call in (True, False):
        run = GpuRun(row_offsets, D, W, B, max(len(idx), 1))
        for name in NAMES:
            getattr(run.bufs, name).zero_()
        run.upload_batch(idx, off, grad)
        run.find_scale()
        run.pack()
        b = run.bufs
        b.cap = cap or b.cap
        for step in range(2):  # (the second finds the workspace and the buffers as the first left them)
            if one_call:
                dq.dqrm_fwd_bwd_step(run.tables, b, run.idx, run.off, run.grad, 0.1, mode)
            else:
                dq.dqrm_embbag_fwd(run.tables, run.idx, run.off, B, mode, b.out, b.codes)
                dq.dqrm_embbag_bwd(run.tables, run.idx, run.off, B, run.grad, b.sorted_pos, b.uniq_rows, b.seg_offsets,
                                   b.table_uniq_offsets, b.num_unique, b.values, b.g_absmax, b.workspace)
                dq.dqrm_grad_quant_int8(b.T, D, b.cap, b.values, b.table_uniq_offsets, b.g_absmax, b.gq, b.g_scale)
                dq.dqrm_sparse_update(run.tables, b.cap, b.uniq_rows, b.table_uniq_offsets, b.gq, b.g_scale, 0.1)
        torch.cuda.synchronize()
        out = {n: getattr(b, n).cpu().numpy() for n in NAMES}
        out["master"], out["packed"], out["status"] = run.master_np(), run.packed_np(), np.array(run.status())
        results.append(out)
    return results


def _compare(a, b):
    for n in a:
        assert_exact(a[n].view(np.uint8), b[n].view(np.uint8), n)


# an empty table among others, an empty batch, bags of none to nine lookups and of one, rows hot enough for many chunks
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("D,B,rows,most", [(16, 128, [1000, 3, 0, 40], 1), (40, 301, [5, 70000, 900], 9), (64, 2048, [2, 3, 500000], 1),
                                           (8, 33, [7], 0), (256, 64, [1], 1)])
def test_one_call_is_its_parts(D, B, rows, most, mode):
    rng = np.random.default_rng(D + B)
    idx, off = _batch(rng, rows, B, lambda T, t, B: np.zeros(B, np.int64) if rows[t] == 0 else
                      rng.integers(0, most + 1, B) if most != 1 else np.ones(B, np.int64))
    grad = (rng.standard_normal((B, len(rows), D)) * 1e-4).astype(np.float32)
    a, b = _runs(rows, D, B, idx, off, grad, mode)
    _compare(a, b)
    assert a["status"][0] == 0 and (len(idx) == 0 or np.abs(a["gq"]).max() == 127)


# Gradients that are not finite: NaN alone; four of them, whose maximum hides those of the same workgroup, beside values far above the
# table's scale, and with nothing but zeros elsewhere (the least scale: quotients that overflow); infinities; a table with none of them.
@pytest.mark.parametrize("D", [16, 64])
def test_one_call_is_its_parts_for_gradients_that_are_not_finite(D):
    rng = np.random.default_rng(D)
    rows, B = [50, 50, 50, 50, 50, 50], 256
    idx, off = _batch(rng, rows, B, lambda T, t, B: np.ones(B, np.int64))
    grad = (rng.standard_normal((B, len(rows), D)) * 1e-4).astype(np.float32)
    grad[3, 0] = np.nan
    grad[5, 1, :4], grad[5, 1, 4:8] = np.nan, 3e38
    grad[:, 2] = 0
    grad[5, 2, :4], grad[5, 2, 4] = np.nan, 3e38
    grad[8, 3, 3] = np.inf
    grad[8, 4, 3], grad[9, 4, 3] = -np.inf, np.nan
    a, b = _runs(rows, D, B, idx, off, grad, 0)
    _compare(a, b)
    large = np.isfinite(a["values"]) & (a["values"] >= np.float32(3e38))
    assert a["g_scale"][2] == np.float32(1e-8) and large.sum() == 5 and (a["gq"][large] == 127).all()
    assert a["status"][0] == 0 and np.isfinite(a["values"][a["table_uniq_offsets"][5]:a["table_uniq_offsets"][6]]).all()


# The edges of the rules that choose the step's launches: tables of as many lookups as one workgroup takes on and one more, a table with far
# more than the others (further ranges; more rows than its workgroup keeps in LDS), rows of one lane group and of a whole wave, and
# bags in more tiles than the forward shares a launch with.
@pytest.mark.parametrize("D,B,rows,lens", [
    (16, 2048, [5000, 2, 300000], 1), (16, 2049, [5000, 2, 300000], 1), (8, 1000, [1000000] + [70] * 15, "one long"),
    (256, 128, [9, 2000, 1], 1), (128, 257, [3000, 50], 1), (64, 8193, [100000, 3], 1), (8, 6200, [900, 5], "ragged"), (24, 40, [4] * 70, "ragged"),
    (40, 1, [7, 1], "ragged"), (8, 3072, [5000, 1, 40], 1), (8, 3073, [5000, 1, 40], 1), (8, 4096, [700, 90, 3] * 11, 1)])
def test_one_call_is_its_parts_at_the_edges_of_its_rules(D, B, rows, lens):
    rng = np.random.default_rng(D + B)
    idx, off = _batch(rng, rows, B, lambda T, t, B: np.ones(B, np.int64) if lens == 1 else rng.integers(0, 5, B) if lens == "ragged"
                      else np.full(B, 20) if t == 0 else rng.integers(0, 2, B))
    grad = (rng.standard_normal((B, len(rows), D)) * 1e-4).astype(np.float32)
    a, b = _runs(rows, D, B, idx, off, grad, 1)
    _compare(a, b)
    assert a["status"][0] == 0


# A row of several chunks whose sum is not finite: NaN in all columns, and in four that one lane holds; beside a row that has the maximum,
# and alone.  (256 lookups: of the narrowest width a workgroup has them all, so that there is one order only.)
@pytest.mark.parametrize("D", [16, 24, 64, 128])
@pytest.mark.parametrize("rows", [1, 2])
@pytest.mark.parametrize("columns", [slice(None), slice(4, 8)], ids=["all", "four"])
def test_one_call_is_its_parts_for_long_rows_that_are_not_finite(columns, rows, D):
    rng = np.random.default_rng(D + rows)
    idx, off = _batch(rng, [rows], 256, lambda T, t, B: np.ones(B, np.int64))
    grad = (rng.standard_normal((256, 1, D)) * 1e-4).astype(np.float32)
    grad[np.flatnonzero(idx == 0)[3], 0, columns] = np.nan
    a, b = _runs([rows], D, 256, idx, off, grad, 0)
    _compare(a, b)
    assert np.isnan(a["values"][0, columns]).all() and a["status"][0] == 0


# The workspace of the one call serves a later segment sum, as a dedupe's does: bags of one lookup and of several (whose chunks a dedupe
# puts in another order), rows of one chunk and of more.
@pytest.mark.parametrize("D,B,rows,bag", [(64, 100, [300, 2, 9], 1), (16, 64, [70] * 12, 4), (40, 33, [5, 70, 900], 3)])
def test_the_workspace_of_one_call_serves_a_segment_sum(D, B, rows, bag):
    import torch

    rng = np.random.default_rng(D + B)
    idx, off = _batch(rng, rows, B, lambda T, t, B: np.full(B, bag))
    grad = (rng.standard_normal((2, B, len(rows), D)) * 1e-4).astype(np.float32)
    ro = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    run = GpuRun(ro, D, np.zeros((ro[-1], D), np.float32), B, len(idx))
    b, dq = run.bufs, run.dq
    run.upload_batch(idx, off, grad[0])
    later = torch.from_numpy(grad[1]).to(run.dev)
    results = []
    for one_call in (True, False):
        if one_call:
            dq.dqrm_fwd_bwd_step(run.tables, b, run.idx, run.off, run.grad, 0.1, 0)
        else:
            dq.dqrm_dedupe(run.tables, run.idx, run.off, B, b.sorted_pos, b.uniq_rows, b.seg_offsets, b.table_uniq_offsets, b.num_unique,
                           b.workspace)
        b.values.zero_()
        for _ in range(2):  # (the first sum's maxima are beside the step's own until it has folded them)
            dq.dqrm_segment_sum(run.tables, B, len(idx), later, b.values, b.g_absmax, b.workspace)
        results.append((b.values.cpu().numpy(), b.g_absmax.cpu().numpy()))
    for x, y, n in zip(*results, ("values", "g_absmax")):
        assert_exact(x.view(np.uint32), y.view(np.uint32), n)
    assert np.abs(results[0][0]).max() > 0 and run.status()[0] == 0


# What the data may have wrong: bad indices at both ends of a table, offsets out of order inside a table, tables whose boundaries go back (and
# so share lookups with others), a batch that does not start at 0 or ends beyond its indices, room for fewer rows than there are, a
# table over the limit.  Nothing is read or written outside a table: everything is as the separate calls leave it.  (16 columns: a workgroup per
# table; 64: three launches.  Of several problems any one is recorded.)
@pytest.mark.parametrize("D,B", [(16, 64), (64, 1024)])
@pytest.mark.parametrize("kind", ["indices", "inside", "boundary", "first", "last", "capacity"])
def test_one_call_is_its_parts_for_bad_batches(kind, D, B):
    import paper_2410_20046_amd as dq

    rng = np.random.default_rng(D + len(kind))
    rows = [50, 3, 900, 7]
    T = len(rows)
    idx, off = _batch(rng, rows, B, lambda T, t, B: np.ones(B, np.int64))
    expected = {dq.ERR_BAD_OFFSETS}
    if kind == "indices":
        for t, bad in enumerate([-1, rows[1], 2 ** 40, rows[3]]):
            idx[t * B], idx[t * B + B - 1], idx[t * B + 9] = bad, bad, -2 ** 40
        expected = {dq.ERR_INDEX_OUT_OF_RANGE}
    elif kind == "inside":
        off[B + 5], off[B + 6], off[3 * B - 4] = off[B + 6], off[B + 5] - 2, off[3 * B - 4] + 30
    elif kind == "boundary":
        off[B] = 2 * B + 7
        expected |= {dq.ERR_INDEX_OUT_OF_RANGE}  # (table 0 has indices of the others)
    elif kind == "first":
        off[0] = -3
    elif kind == "last":
        off[T * B] = T * B + 9
    grad = (rng.standard_normal((B, T, D)) * 1e-4).astype(np.float32)
    print(f"bad batch: {kind}, {T} tables x {B} x {D}", flush=True)
    a, b = _runs(rows, D, B, idx, off, grad, 1, cap=60 if kind == "capacity" else None)
    status = a.pop("status"), b.pop("status")
    _compare(a, b)
    assert all(s[0] == 0 if kind == "capacity" else s[0] in expected for s in status), status
    assert a["num_unique"][0] > 60 or kind != "capacity"


def test_one_call_is_its_parts_for_a_table_over_the_limit():
    import paper_2410_20046_amd as dq

    T, B, D = 35, 2000, 8
    rng = np.random.default_rng(1)
    idx, off = _batch(rng, [900] * T, B, lambda T, t, B: np.full(B, T if t == 0 else 0))
    grad = (rng.standard_normal((B, T, D)) * 1e-4).astype(np.float32)
    a, b = _runs([900] * T, D, B, idx, off, grad, 1)
    assert a.pop("status")[0] == b.pop("status")[0] == dq.ERR_CAPACITY
    _compare(a, b)
    assert a["num_unique"][0] == 0
