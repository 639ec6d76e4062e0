"""dqrm_dedupe at the sizes where its split of a table's rows into ranges changes hands: the table sizes around the ranges
(fewer rows than ranges, one row, a hot row that overflows what a workgroup sorts in LDS), the lookups per table at which
another workgroup size or the tile-by-tile partition takes over, bags of equal and unequal length and more bags than fit the
LDS, bad indices at every kind of place.  Everything is an integer: exact equality with the oracle, except where indices are
bad, which the oracle does not take (numpy's stable sort then)."""
import numpy as np
import pytest

from gen import Workload
from helpers import GpuRun, assert_exact

pytestmark = pytest.mark.gpu


def _dedupe(wl, idx, off, B):
    run = GpuRun(wl.row_offsets, wl.D, np.zeros((wl.R, wl.D), np.float32), B, len(idx), with_packed=False, want_codes=False)
    run.upload_batch(idx, off)
    b = run.bufs
    b.workspace.fill_(0xA5)  # (whatever is in it)
    run.dq.dqrm_dedupe(run.tables, run.idx, run.off, B, b.sorted_pos, b.uniq_rows, b.seg_offsets, b.table_uniq_offsets,
                       b.num_unique, b.workspace)
    U = int(b.num_unique.cpu().item())
    return run, dict(U=np.array([U]), sorted_pos=b.sorted_pos.cpu().numpy()[:len(idx)], uniq_rows=b.uniq_rows.cpu().numpy()[:U],
                     seg_offsets=b.seg_offsets.cpu().numpy()[:U + 1], table_uniq_offsets=b.table_uniq_offsets.cpu().numpy())


def _expected(wl, idx, off, B):
    """From the definition: a stable sort by (table, row), bad rows last in their table and in no segment."""
    pos, rows, seg, tuo = [], [], [], [0]
    for t in range(wl.T):
        lo, hi = int(off[t * B]), int(off[(t + 1) * B])
        v, n = idx[lo:hi], int(wl.cards[t])
        key = np.where((v < 0) | (v >= n), n, v)
        order = np.argsort(key, kind="stable")
        k = key[order]
        heads = np.flatnonzero((k < n) & (np.concatenate([[-1], k[:-1]]) != k))
        pos.append(lo + order)
        rows.append(k[heads])
        seg.append(lo + heads)
        tuo.append(tuo[-1] + len(heads))
    cat = np.concatenate
    return dict(U=np.array([tuo[-1]]), sorted_pos=cat(pos).astype(np.int32), uniq_rows=cat(rows).astype(np.int64),
                seg_offsets=cat(seg + [[len(idx)]]).astype(np.int32), table_uniq_offsets=np.array(tuo, np.int32))


# lookups per table; tables: one row, fewer rows than ranges, as many as a digit has values and one more, many
@pytest.mark.parametrize("n", [1, 63, 512, 513, 2047, 4096, 4097, 8192, 8193, 16384, 16385, 65535, 65536])
@pytest.mark.parametrize("cards", [(1, 3, 255, 40), (256, 257, 7_000_003)], ids=["tiny", "large"])
def test_lookups_per_table(n, cards):
    cards = np.array(cards, np.int64)
    T = len(cards)
    wl = Workload(name="ranges", T=T, D=8, B=n, alpha=1.05, seed=n + T, cards=cards)
    idx, off = wl.batch(0)
    print(f"ranges: {n} lookups in each of {cards.tolist()}", flush=True)
    run, got = _dedupe(wl, idx, off, n)
    for k, v in _expected(wl, idx, off, n).items():
        assert_exact(got[k], v, f"n={n} {k}")
    assert run.status()[0] == 0


# Ranges chosen by a sample: rows that take several ranges' share, close together, at either end, one row alone, all
# alike; more in one range than a workgroup holds although the sample shows nothing of it (every 256th lookup is what the sample sees);
# and beside them tables of fewer lookups than the sample has, and of none, and bad indices.
@pytest.mark.parametrize("T", [1, 6])
@pytest.mark.parametrize("kind", ["spread", "one row", "two rows", "cluster", "ends", "unseen"])
def test_ranges_by_a_sample(kind, T):
    rng = np.random.default_rng(len(kind) + T)
    n, rows = 65_536, 3_000_000
    lens = [n] + [0, 40, 17_001, 65_535, n][:T - 1]
    cards = np.array([rows, 9, 70, 1, 65_536, rows][:T], np.int64)
    idx = []
    for c, m in zip(cards, lens):
        v = rng.integers(0, c, m)
        hot = rng.random(m) < 0.9
        if kind == "one row":
            v[:] = c // 2
        elif kind == "two rows":
            v = np.where(rng.random(m) < 0.5, c - 1, c // 3)
        elif kind == "cluster":
            v = np.where(hot, np.minimum(c // 5 + rng.integers(0, 40, m), c - 1), v)
        elif kind == "ends":
            v = np.where(hot, np.where(rng.random(m) < 0.5, 0, c - 1), v)
        elif kind == "unseen":
            v = np.where(np.arange(m) % 256 != 0, v // 100, v)
        v[rng.integers(0, max(m, 1), m // 1000)] = rng.choice([-1, c, 2 ** 40])
        idx.append(v)
    idx, B = np.concatenate(idx).astype(np.int64), 512
    starts = np.concatenate([[0], np.cumsum(lens)])
    off = np.concatenate([np.sort(rng.integers(0, m + 1, B)) + s for m, s in zip(lens, starts)] + [[len(idx)]]).astype(np.int64)
    off[np.arange(T) * B] = starts[:T]
    wl = Workload(name="sample", T=T, D=8, B=B, alpha=1.0, seed=1, cards=cards)
    print(f"sampled ranges: {kind}, {T} tables", flush=True)
    run, got = _dedupe(wl, idx, off, B)
    for k, v in _expected(wl, idx, off, B).items():
        assert_exact(got[k], v, f"{kind} {k}")
    assert run.status()[0] == run.dq.ERR_INDEX_OUT_OF_RANGE


# The rules of partitioned tables: from two tiles per table on, with few tables from three; a workgroup that sorts 4096, or, where there is
# a CU for each or a range has many lookups, 8192.  Beside each other tables that are cut into ranges of equal width (evenly spread
# lookups, fewer rows than ranges, a few more) and by the sample (popular rows, at one end, a single row among many), bad indices in some.
@pytest.mark.parametrize("T,n", [(5, 16_384), (5, 16_385), (4, 24_576), (4, 24_577), (8, 16_385), (9, 30_011), (9, 65_536), (100, 27_000), (128, 16_391)])
def test_partitioned_tables_of_all_kinds(T, n):
    rng = np.random.default_rng(T + n)
    cards, idx = [], []
    for t in range(T):
        c = [900_000, 20, 33, 70_000, 5_000_000, 1_000, 40, 3][t % 8]
        v = rng.integers(0, c, n)
        if t % 8 == 3:  # popular rows all over the table
            v = (np.minimum(rng.zipf(1.1, n), c) * 7919) % c
        elif t % 8 == 4:
            v = np.where(rng.random(n) < 0.8, np.minimum(rng.zipf(1.3, n), c) - 1, v)
        elif t % 8 == 5:
            v = np.where(rng.random(n) < 0.6, c // 2, v)
        if t % 3 == 1:
            v[rng.integers(0, n, 5)] = rng.choice([-1, c, 2 ** 40], 5)
        cards.append(c)
        idx.append(v)
    wl = Workload(name="kinds", T=T, D=8, B=n, alpha=1.0, seed=1, cards=np.array(cards, np.int64))
    idx, off = np.concatenate(idx).astype(np.int64), np.arange(T * n + 1, dtype=np.int64)
    print(f"partitioned: {T} tables of {n} lookups", flush=True)
    run, got = _dedupe(wl, idx, off, n)
    for k, v in _expected(wl, idx, off, n).items():
        assert_exact(got[k], v, f"T={T} n={n} {k}")
    assert run.status()[0] == run.dq.ERR_INDEX_OUT_OF_RANGE


@pytest.mark.parametrize("n", [400, 3000, 8000, 40000])
@pytest.mark.parametrize("bags", ["ragged", "pairs", "sparse"])
def test_hot_rows_and_bags(n, bags):
    """One table with nearly all of the batch's lookups, most of them to one row at the front, in the middle or at the end of
    its rows; the bags of unequal length, of two lookups (twice the batch's average, so they are searched for all the same) and
    many more than the lookups."""
    T, big = 3, min(3 * n - 2, 65536)
    rng = np.random.default_rng(n + len(bags))
    B = {"ragged": 777, "pairs": (big + 1) // 2, "sparse": 20011}[bags]
    cards = np.array([2000, 50, 100_000], np.int64)
    for hot in (0, 49_999, 99_999):
        if bags == "pairs":
            lens = np.full(B, 2, np.int64)
        else:
            lens = np.bincount(rng.integers(0, B, big), minlength=B).astype(np.int64)
        lens = np.concatenate([(np.arange(B) == 0), (np.arange(B) == B - 1), lens]).astype(np.int64)
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        m = int(off[-1]) - 2
        last = rng.integers(0, 100_000, m)
        last[rng.random(m) < 0.7] = hot
        last[rng.random(m) < 0.2] = min(hot + 1, 99_999)
        last[rng.random(m) < 0.01] = 100_000  # bad: past the end
        last[rng.random(m) < 0.01] = -7
        idx = np.concatenate([[1999], [0], last]).astype(np.int64)
        wl = Workload(name="hot", T=T, D=8, B=B, alpha=1.05, seed=1, cards=cards)
        print(f"hot row {hot}, {m} lookups in {B} bags ({bags})", flush=True)
        run, got = _dedupe(wl, idx, off, B)
        for k, v in _expected(wl, idx, off, B).items():
            assert_exact(got[k], v, f"n={n} hot={hot} {bags} {k}")
        code, tb, val = run.status()
        assert code == run.dq.ERR_INDEX_OUT_OF_RANGE and tb == 2 and val in (100_000, -7)
        # the bags reach the segment sums: gradients that name their bag (sums of integers below 2^24, exact)
        g = np.zeros((B, T, 8), np.float32)
        g[:, 2, 0] = np.arange(B) % 251
        run.upload_batch(idx, off, g)
        b = run.bufs
        run.dq.dqrm_segment_sum(run.tables, B, len(idx), run.grad, b.values, b.g_absmax, b.workspace)
        bag = np.repeat(np.arange(B), np.diff(off[2 * B:]))
        good = (last >= 0) & (last < 100_000)
        want = np.bincount(last[good], weights=(bag[good] % 251).astype(np.float64), minlength=100_000)
        s0 = int(got["table_uniq_offsets"][2])
        rows = got["uniq_rows"][s0:]
        assert_exact(b.values.cpu().numpy()[s0:s0 + len(rows), 0].astype(np.float64), want[rows], f"n={n} hot={hot} {bags} sums")


# Every table has as many lookups as if all bags of the batch were equally long, and the bag of a lookup is guessed from that: rightly
# (`equal`) or wrongly (half of the bags one longer, the others one shorter; one bag empty and one twice as long).  Sizes for each of
# the workgroups, a range that overflows the LDS, tables sorted by tiles; a row with most of the lookups or none.
@pytest.mark.parametrize("n", [400, 3000, 8000, 13_000, 40_000, 65_535])
@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("bags", ["equal", "halves", "one off"])
def test_bags_that_add_up(n, T, bags):
    rng = np.random.default_rng(n + T)
    B = n // 5
    lens = np.full((T, B), 5, np.int64)
    if bags == "halves":
        lens[:, : B // 2] += 1
        lens[:, B - B // 2:] -= 1
    elif bags == "one off":
        lens[:, B // 3] = 0
        lens[:, B // 2] = 10
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1))]).astype(np.int64)
    cards = np.full(T, 50_000, np.int64)
    wl = Workload(name="add up", T=T, D=8, B=B, alpha=1.05, seed=1, cards=cards)
    for hot in (0.0, 0.75):
        idx = rng.integers(0, 50_000, int(off[-1]))
        idx[rng.random(len(idx)) < hot] = 31_234
        print(f"{T} tables of {5 * B} lookups, bags {bags}, hot {hot}", flush=True)
        run, got = _dedupe(wl, idx, off, B)
        for k, v in _expected(wl, idx, off, B).items():
            assert_exact(got[k], v, f"n={n} T={T} {bags} hot={hot} {k}")
        _sums_exact(run, idx, off, B, cards, got, f"n={n} T={T} {bags} hot={hot}")
        assert run.status()[0] == 0


# Boundaries between tables that go backwards: the table that ends before it begins is reported and skipped, and so is a later one
# that has lookups of an earlier one (the distinct rows would outgrow the outputs otherwise).  Tables per kind of lookup for such a
# boundary: one step of a workgroup, several; lookups for the plain and the partitioned sort.
@pytest.mark.parametrize("T,n,B", [(4, 100, 10), (5, 40_000, 500), (100, 60, 7), (700, 30, 3)])
def test_tables_that_share_lookups(T, n, B):
    bound = np.arange(T + 1, dtype=np.int64) * n
    bound[T - 2:] -= n // 2  # table T - 3 ends where it began less half a table; T - 2 shares that half with T - 4
    bound[T - 2:] -= n
    if T > 4:
        bound[1], bound[2] = n + n // 3, n + n // 4  # and table 1 ends before it begins; table 2 shares a few with table 0
    N = int(bound.max())
    off = np.concatenate([np.linspace(bound[t], bound[t + 1], B + 1)[:-1].astype(np.int64) for t in range(T)] + [bound[-1:]])
    cards = np.full(T, 40, np.int64)
    idx = np.random.default_rng(T).integers(0, 40, N).astype(np.int64)
    keep = []
    for t in range(T):
        lo, hi = int(bound[t]), int(bound[t + 1])
        sane = [(int(bound[s]), int(bound[s + 1])) for s in range(t) if bound[s] <= bound[s + 1]]
        keep.append(lo <= hi and not any(l < hi and lo < h for l, h in sane))
    assert 0 < sum(keep) < T - 1
    print(f"shared lookups: {T} tables, {sum(keep)} kept, {N} lookups", flush=True)
    wl = Workload(name="shared", T=T, D=8, B=B, alpha=1.05, seed=1, cards=cards)
    spare = 4096
    run = GpuRun(wl.row_offsets, 8, np.zeros((wl.R, 8), np.float32), B, N + spare, with_packed=False, want_codes=False)
    run.upload_batch(idx, off)
    b, dq = run.bufs, run.dq
    for x in (b.sorted_pos, b.uniq_rows, b.seg_offsets):
        x.fill_(-9)
    b.workspace.fill_(0xA5)
    dq.dqrm_dedupe(run.tables, run.idx, run.off, B, b.sorted_pos, b.uniq_rows, b.seg_offsets, b.table_uniq_offsets, b.num_unique,
                   b.workspace)
    pos, rows, tuo = np.full(N + spare, -9, np.int32), [], [0]
    for t in range(T):
        lo, hi = int(bound[t]), int(bound[t + 1])
        u = np.zeros(0, np.int64)
        if keep[t]:
            pos[lo:hi] = lo + np.argsort(idx[lo:hi], kind="stable")
            u = np.unique(idx[lo:hi])
        rows.append(u)
        tuo.append(tuo[-1] + len(u))
    U = tuo[-1]
    assert int(b.num_unique.cpu().item()) == U
    assert_exact(b.table_uniq_offsets.cpu().numpy(), np.array(tuo, np.int32), "table_uniq_offsets")
    assert_exact(b.sorted_pos.cpu().numpy(), pos, "sorted_pos")
    got = b.uniq_rows.cpu().numpy()
    assert_exact(got[:U], np.concatenate(rows), "uniq_rows")
    assert (got[U:] == -9).all() and (b.seg_offsets.cpu().numpy()[U + 1:] == -9).all()
    used = dq.dqrm_embbag_bwd_workspace_bytes(T, 8, B, N)
    assert (b.workspace[used:] == 0xA5).all().item()
    assert run.status()[0] == dq.ERR_BAD_OFFSETS


def _sums_exact(run, idx, off, B, cards, got, what):
    """The bags and the chunk lists, through the segment sums: gradients that name their bag (sums of integers below 2^24, exact)."""
    T = len(cards)
    g = np.zeros((B, T, 8), np.float32)
    g[:, :, 0] = np.arange(B)[:, None] % 61
    run.upload_batch(idx, off, g)
    b = run.bufs
    run.dq.dqrm_segment_sum(run.tables, B, len(idx), run.grad, b.values, b.g_absmax, b.workspace)
    values = b.values.cpu().numpy()[:int(got["U"][0]), 0].astype(np.float64)
    for t in range(T):
        lo, hi = int(off[t * B]), int(off[(t + 1) * B])
        v, bag = idx[lo:hi], np.repeat(np.arange(B), np.diff(off[t * B:(t + 1) * B + 1]))
        good = (v >= 0) & (v < cards[t])
        want = np.bincount(v[good], weights=(bag[good] % 61).astype(np.float64), minlength=int(cards[t]))
        s, e = got["table_uniq_offsets"][t:t + 2]
        assert_exact(values[s:e], want[got["uniq_rows"][s:e]], f"{what} sums of table {t}")


def _uneven(seed, per_table, cards, B, alike, hot=None, bad=0.0):
    """A batch with per_table[t] lookups of table t: bags of random lengths, or (alike) as equal as they can be; popular rows
    first in every table, and `hot` of a large table's lookups to one of its rows."""
    rng = np.random.default_rng(seed)
    idx, lens = [], []
    for n, r in zip(per_table, cards):
        v = np.minimum((rng.random(n) ** 4 * r).astype(np.int64), r - 1)
        if n > 4096:
            if hot:
                v[rng.random(n) < hot] = r // 3
            v[rng.random(n) < bad] = r + 5
            v[rng.random(n) < bad] = -1
        idx.append(v)
        lens.append(np.diff(np.arange(B + 1) * n // B) if alike else np.bincount(rng.integers(0, B, n), minlength=B))
    off = np.concatenate([[0], np.cumsum(np.concatenate(lens))]).astype(np.int64)
    return np.concatenate(idx).astype(np.int64), off


# Tables with far more lookups than the others: their further ranges and the order of all ranges, at each of the workgroups, for
# one such table and several (first, last, neighbours), with few rows, a hot row and bad indices; up to the most tables.
@pytest.mark.parametrize("per_table,B", [
    ([128] * 40 + [65536] + [3000] + [128] * 3, 128), ([65536] + [1] * 1023, 16), ([100] * 300 + [2049, 4097, 20_000], 100),
    ([2048] * 25 + [65536], 512), ([16_385] + [2048] * 12 + [30_000, 30_000], 700), ([65536, 1, 2, 65536], 8192),
    ([8192] * 12 + [40_000, 37_000, 65536], 3000), ([9000] * 20 + [65535], 9000), ([600] * 1000 + [40_000, 50_000], 600)])
@pytest.mark.parametrize("kind", ["plain", "hot", "few"])
def test_uneven_tables(per_table, B, kind):
    T = len(per_table)
    cards = np.where(np.array(per_table) > 4096, {"plain": 200_000, "hot": 5000, "few": 7}[kind], 300).astype(np.int64)
    idx, off = _uneven(T, per_table, cards, B, kind == "plain", hot=0.6 if kind == "hot" else None, bad=0.02 if kind == "hot" else 0.0)
    wl = Workload(name="uneven", T=T, D=8, B=B, alpha=1.05, seed=1, cards=cards)
    print(f"uneven: {T} tables of up to {max(per_table)} lookups ({kind})", flush=True)
    run, got = _dedupe(wl, idx, off, B)
    for k, v in _expected(wl, idx, off, B).items():
        assert_exact(got[k], v, f"{kind} {k}")
    _sums_exact(run, idx, off, B, cards, got, kind)
    assert (run.status()[0] != 0) == (kind == "hot")


def _dedupe_batches(data, cards, B, bound=0):
    """The batches (indices, offsets) in one launch, checked against _expected and through the segment sums."""
    T = len(cards)
    wl = Workload(name="batches", T=T, D=8, B=B, alpha=1.05, seed=1, cards=cards)
    most = max(len(i) for i, _ in data)
    runs = []
    for idx, off in data:
        run = GpuRun(wl.row_offsets, 8, np.zeros((wl.R, 8), np.float32), B, most, with_packed=False, want_codes=False)
        run.upload_batch(idx, off)
        run.bufs.workspace.fill_(0xA5)
        runs.append(run)
    b = [r.bufs for r in runs]
    runs[0].dq.dqrm_dedupe_multi(runs[0].tables, B, [(r.idx, r.off, x.sorted_pos, x.uniq_rows, x.seg_offsets, x.table_uniq_offsets,
                                                      x.num_unique, x.workspace) for r, x in zip(runs, b)], max_table_lookups=bound)
    for (idx, off), r, x in zip(data, runs, b):
        U = int(x.num_unique.cpu().item())
        got = dict(U=np.array([U]), sorted_pos=x.sorted_pos.cpu().numpy()[:len(idx)], uniq_rows=x.uniq_rows.cpu().numpy()[:U],
                   seg_offsets=x.seg_offsets.cpu().numpy()[:U + 1], table_uniq_offsets=x.table_uniq_offsets.cpu().numpy())
        for k, v in _expected(wl, idx, off, B).items():
            assert_exact(got[k], v, k)
        _sums_exact(r, idx, off, B, cards, got, "batch")
    return runs[0].status()


# Batches of one launch: their tables' sizes differ from batch to batch; partitioned ones; more tables than are ever partitioned.
@pytest.mark.parametrize("batches", [
    [[128] * 30, [128] * 29 + [60_000], [60_000] + [1] * 29], [[17_000, 16_500, 20_000], [65536, 16_400, 10_000]],
    [[16_500] * 140]], ids=["uneven", "partitioned", "many"])
def test_batches_of_one_launch(batches):
    T, B = len(batches[0]), 900
    cards = np.full(T, 3000, np.int64)
    print(f"batches of {[sum(p) for p in batches]} lookups in {T} tables", flush=True)
    status = _dedupe_batches([_uneven(k, p, cards, B, False) for k, p in enumerate(batches)], cards, B)
    assert status[0] == 0


# A launch of so many tables that each is one workgroup's (64 tables x 2 batches, more than 2048 lookups in the average table, at
# most 16384 in any): lookups at the edges of a workgroup's rounds, tables of one row to many bits of row, hot rows and bad indices,
# bags of one lookup, of unequal length, unequal but adding up as if equal, and more bags than the LDS holds.
@pytest.mark.parametrize("bags", ["one", "ragged", "pretend", "many"])
@pytest.mark.parametrize("rows", [1, 2, 255, 256, 70_000])
def test_whole_tables(bags, rows):
    T = 64
    cards = np.full(T, min(rows, 3000), np.int64)
    cards[[0, 9, T - 1]] = rows
    data = []
    if bags in ("one", "pretend"):  # every table has as many lookups
        B = {"one": 16384, "pretend": 1500}[bags] if rows != 256 else 2051
        per_table = [B * (1 if bags == "one" else 5)] * T
    else:
        B = {"ragged": 700, "many": 20_001}[bags]
        per_table = [0, 1, 2, 63, 64, 65, 1023, 1024, 1025, 16384, 16383, 15_361] + [2500] * (T - 12)
    for k in range(2):
        idx, off = _uneven(k, per_table, cards, B, bags in ("one", "pretend"), hot=0.3 if k else None, bad=0.01 * k)
        if bags == "pretend":
            lens = np.full((T, B), 5)
            lens[:, : B // 2] += 1
            lens[:, B - B // 2:] -= 1
            off = np.concatenate([[0], np.cumsum(lens.reshape(-1))]).astype(np.int64)
        data.append((idx, off))
    print(f"whole tables: {bags}, {B} bags, {rows} rows, {max(per_table)} lookups", flush=True)
    status = _dedupe_batches(data, cards, B, bound=16384)
    assert status[0] == (0 if max(per_table) <= 4096 else -4)
