"""The work that a user of this package has it do, as timed cases.

A case is one pass through the public entry points on tables, batches and (where the dense part belongs to it) MLPs of
the shapes the repository's configurations name, plus ragged and odd shapes of the same ranges:

  step     one training step of the embedding layer: forward, dedupe, segment sums, INT8 codes, sparse update
  ahead    several such steps, their batches deduplicated in one launch before them (a data loader has the indices)
  serve    the forward alone
  train    the full train step: forward, MLPs + interaction + loss + their backward and SGD, backward, update
  nodes    one weight update from several micro-batches (simulated data parallelism)
  refresh  the per-table scales recomputed from the whole tables and the packed mirror re-encoded

`calls` says which of the equivalent call sequences a step takes: "five" is dqrm_fwd_bwd_step (forward, backward,
INT8 codes, update: what a caller takes who exchanges the codes), "one_pass" ends in dqrm_quant_update.
`pooling` / `bag`: "one" lookup per bag, "fixed" = `bag` lookups in each, "ragged" = 0 .. `bag` lookups.
"""
from __future__ import annotations

import math
from typing import Dict, List

import numpy as np
import torch

import paper_2410_20046_amd as dq

LR = 0.1
TRAIN_LR = 1e-3  # of the full step: small enough that every drawn model trains (0.1 lets some diverge within a few passes)
ROW_MIN, ROW_MAX = 3, 10_000_000  # table sizes: log-uniform in this range, as in the Criteo-shaped workloads
KAGGLE = dict(T=26, D=16, rows=33_770_000, alpha=1.05)
TERABYTE = dict(T=26, D=64, rows=49_120_000, alpha=1.1)
# MLP widths of the two models; the bottom MLP ends at the embedding width, the top MLP starts at the interaction's
KAGGLE_MLP = dict(num_dense=13, bot="512-256-64", top="512-256")
TERABYTE_MLP = dict(num_dense=13, bot="512-256", top="512-512-256")


def listed() -> List[dict]:
    one = dict(pooling="one", bag=1)
    return [
        # the smallest step: all launches and latency (the "tiny" configuration: 1000 rows per table, uniform indices)
        dict(name="tiny step", kind="step", T=4, D=16, rows=4000, even=True, alpha=0.0, B=128, mode="master", calls="five", **one),
        # the two model shapes, a step of the tables alone, every call in line
        dict(name="kaggle step", kind="step", **KAGGLE, B=2048, mode="packed", calls="five", **one),
        dict(name="terabyte step", kind="step", **TERABYTE, B=8192, mode="packed", calls="one_pass", **one),
        # the benchmark's default: the sort of the next 8 batches in one launch, then their 8 steps
        dict(name="terabyte ahead", kind="ahead", **TERABYTE, B=8192, mode="packed", steps=8, **one),
        # multi-hot features with empty bags at sizes that fit no tile; the largest batch a table's lookup limit allows
        dict(name="ragged bags", kind="step", T=13, D=40, rows=2_345_678, alpha=1.05, B=3001, mode="master", calls="five",
             pooling="ragged", bag=7),
        dict(name="pooled step", kind="step", **TERABYTE, B=8192, mode="packed", calls="one_pass", pooling="fixed", bag=8),
        # inference: a small request and a large multi-hot one
        dict(name="serve small", kind="serve", **KAGGLE, B=32, mode="packed", **one),
        dict(name="serve large", kind="serve", **TERABYTE, B=8192, mode="packed", pooling="ragged", bag=8),
        # the full train step of both models; the second with INT4 MLP weights and INT8 MLP gradients
        dict(name="train kaggle", kind="train", **KAGGLE, B=2048, mode="packed", wbits=0, gbits=0, **KAGGLE_MLP, **one),
        dict(name="train terabyte quantised", kind="train", **TERABYTE, B=8192, mode="packed", wbits=4, gbits=8, **TERABYTE_MLP, **one),
        # eight micro-batches of 1024, one update
        dict(name="simulated nodes", kind="nodes", **TERABYTE, B=8192, mode="packed", nodes=8, **one),
        # the periodic scale refresh over the whole tables
        dict(name="scale refresh", kind="refresh", **TERABYTE),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["step", "step", "step", "ahead", "serve", "train", "train", "nodes", "refresh"])
    D = rng.choice([8, 16, 16, 24, 32, 40, 64, 64, 72, 128, 256])
    T = _log_int(rng, 1, 60 if kind != "train" else 50)
    if kind == "train":
        D = rng.choice([8, 16, 16, 24, 32, 64])
        T = min(T, 4096 // D - 1)
    rows = min(_log_int(rng, max(3 * T, 1000), 50_000_000), T * ROW_MAX, 3_140_000_000 // D)
    case = dict(kind=kind, T=T, D=D, rows=rows, alpha=rng.choice([0.0, 1.05, 1.1, 1.2]))
    if kind == "refresh":
        return case
    case["mode"] = rng.choice(["packed", "packed", "master"])
    case["pooling"] = rng.choice(["one", "one", "fixed", "ragged"])
    case["bag"] = 1 if case["pooling"] == "one" else rng.randint(2, 8)
    # samples: no more gradient bytes than the Terabyte shape's, no more lookups than its pooled step's
    most = min(16384, 26 * 8192 * 64 // (T * D), 26 * 65536 // (T * case["bag"]), 65536 // case["bag"])
    B = _log_int(rng, min(16, most), most)
    if kind == "step":
        case["calls"] = rng.choice(["five", "one_pass"])
    elif kind == "ahead":
        case["steps"] = rng.randint(2, 8)
        B = max(1, B * 2 // case["steps"]) if case["bag"] > 1 else B
    elif kind == "nodes":
        case["nodes"] = rng.randint(2, 8)
        B = max(1, B // case["nodes"]) * case["nodes"]
    elif kind == "train":
        case["wbits"], case["gbits"] = rng.choice([(0, 0), (0, 0), (4, 8), (4, 0), (0, 8)])
        case["num_dense"] = rng.randint(4, 20)
        width = lambda: 4 * rng.randint(12, 128) + rng.choice([0, 0, 0, 1])  # noqa: E731
        case["bot"] = "-".join(str(width()) for _ in range(rng.randint(1, 3)))
        case["top"] = "-".join(str(width()) for _ in range(rng.randint(1, 3)))
        B = min(B, 8192)
    case["B"] = B
    return case


# ---- shapes -----------------------------------------------------------------------------------------------------


def table_rows(case: dict) -> np.ndarray:
    """Rows of each table: evenly spaced quantiles of the log-uniform distribution, scaled to the total with a cap."""
    T, total = case["T"], case["rows"]
    if case.get("even"):
        return np.full(T, total // T, dtype=np.int64)
    c = np.exp(math.log(ROW_MIN) + (np.arange(T) + 0.5) / T * (math.log(ROW_MAX) - math.log(ROW_MIN)))
    for _ in range(64):
        c = np.clip(c, ROW_MIN, ROW_MAX)
        free = c < ROW_MAX
        if not free.any() or abs(c.sum() - total) < 0.5:
            break
        c[free] *= max(total - c[~free].sum(), ROW_MIN) / c[free].sum()
    return np.clip(np.rint(c), ROW_MIN, ROW_MAX).astype(np.int64)


def lookups_per_table(case: dict) -> float:
    return case["B"] * (case["bag"] / 2 if case["pooling"] == "ragged" else case["bag"])


def expected_unique(case: dict, lookups: float) -> float:
    """Distinct rows that `lookups` draws per table touch, on average, over all tables."""
    total = 0.0
    for r in table_rows(case):
        edges = np.unique(np.concatenate([np.arange(1, min(int(r), 1024) + 1), np.geomspace(1, int(r), 400).astype(np.int64), [int(r) + 1]]))
        count = np.diff(edges)
        weight = (edges[:-1] + (count - 1) / 2.0) ** -case["alpha"]
        p = np.minimum(weight / (weight * count).sum(), 1 - 1e-12)
        total += float((count * -np.expm1(lookups * np.log1p(-p))).sum())
    return total


def mlp_dims(case: dict):
    V = case["T"] + 1
    hidden = lambda key: [int(w) for w in case[key].split("-")]  # noqa: E731
    return ([case["num_dense"]] + hidden("bot") + [case["D"]],
            [case["D"] + V * (V - 1) // 2] + hidden("top") + [1])


def work(case: dict) -> Dict[str, float]:
    T, D, kind = case["T"], case["D"], case["kind"]
    R = int(table_rows(case).sum())
    if kind == "refresh":  # the scale has to be known before the first code: the tables are read twice
        return {"bytes": 2 * 4 * D * R + D / 2 * R, "flops": 0}
    B = case["B"]
    bags, N = T * B, T * lookups_per_table(case)
    packed = case["mode"] == "packed"
    steps = case.get("steps", 1)
    # (a batch's distinct rows are read once, whatever the step does with them)
    U = expected_unique(case, lookups_per_table(case))
    ids = 8 * N + 8 * bags
    if kind == "serve":
        return {"bytes": ids + (D / 2 if packed else 4 * D) * U + 4 * D * bags, "flops": 2 * N * D}
    read = 4 * D * U + (D / 2 * U if packed else 0)
    write = 4 * D * bags + (4 * N + 12 * U) + 4 * D * U + D * U + 4 * D * U + D / 2 * U
    if kind == "nodes":
        per_node = expected_unique(case, lookups_per_table(case) / case["nodes"]) * case["nodes"]
        # the blocks' rows, values and codes, then the merged rows and their 32-bit sums
        write = 4 * D * bags + 4 * N + per_node * (12 + 5 * D) + U * (8 + 4 * D) + 4 * D * U + D / 2 * U
        ids *= 2  # the micro-batches' own index lists beside the whole batch's
    step = {"bytes": ids + read + 4 * D * bags + write, "flops": 4 * N * D}
    if kind == "train":
        bot, top = mlp_dims(case)
        weights = sum(i * o for d in (bot, top) for i, o in zip(d[:-1], d[1:]))
        pairs = (T + 1) * T // 2
        state = 4 * weights * 2 + (9 * weights if case["gbits"] else 0)
        step["bytes"] += B * 4 * (case["num_dense"] + 1) + state
        step["flops"] += 6 * B * weights - 2 * B * bot[0] * bot[1] + 6 * B * pairs * D
    return {k: v * steps for k, v in step.items()}


def tolerance(case: dict):
    # The tables' path has a documented order of every sum: integers and floats are the same bits, whoever computes
    # them.
    if case["kind"] != "train":
        return "exact"
    # The dense part's products may be added in any order.  Against the same steps with the dense part in float64 most
    # outputs agree to 1e-6; but a pre-activation within rounding of zero flips its ReLU's derivative and a value within
    # rounding of a code's edge flips the code.  Seen over three steps of 80 drawn models: 8.3e-4 of the 2-norm, 0.27 at
    # one element (embedding gradients of the sample concerned), 4.5e-4 of an array of codes; about four times that:
    return {"rel": 3e-3, "max": 0.9, "differ": 2e-3}


# ---- inputs -----------------------------------------------------------------------------------------------------


class Draws:
    """Seeded inputs on the GPU."""

    def __init__(self, case: dict, seed: int):
        self.case, self.dev = case, torch.device("cuda:0")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(seed * 7919 + 12345)
        self.rows = table_rows(case)
        self.shift = torch.randint(0, ROW_MAX, (case["T"],), generator=self.g, device=self.dev).tolist()

    def tables(self) -> dq.Tables:
        """Tables U(-1/sqrt(rows), 1/sqrt(rows)) with their scales and packed mirror, as training starts."""
        offsets = np.concatenate([[0], np.cumsum(self.rows)]).astype(np.int64)
        R, D = int(offsets[-1]), self.case["D"]
        master = torch.empty((R, D), dtype=torch.float32, device=self.dev)
        for t, r in enumerate(self.rows):
            b = 1.0 / math.sqrt(int(r))
            master[offsets[t]:offsets[t + 1]].uniform_(-b, b, generator=self.g)
        packed = torch.zeros((R, D // 2), dtype=torch.uint8, device=self.dev)
        tables = dq.Tables(offsets, D, master, packed)
        dq.dqrm_find_scale(tables)
        dq.dqrm_pack_int4(tables)
        return tables

    def lengths(self, B: int) -> torch.Tensor:
        c = self.case
        if c["pooling"] == "ragged":  # each length equally often (so every batch has as many lookups), in random order
            order = torch.rand((c["T"], B), generator=self.g, device=self.dev).argsort(dim=1)
            return order % (c["bag"] + 1)
        return torch.full((c["T"], B), c["bag"], dtype=torch.int64, device=self.dev)

    def batches(self, count: int, B: int):
        """`count` batches (indices, offsets), table-major; row popularity is Zipf(alpha), hot rows scattered."""
        lens = [self.lengths(B) for _ in range(count)]
        per_table = torch.stack([x.sum(dim=1) for x in lens]).tolist()  # [count][T]
        parts: List[List[torch.Tensor]] = [[] for _ in range(count)]
        for t, r in enumerate(int(x) for x in self.rows):
            if self.case["alpha"] > 0:
                cdf = torch.cumsum(torch.arange(1, r + 1, dtype=torch.float64, device=self.dev) ** -self.case["alpha"], 0)
                cdf /= cdf[-1].clone()
            for k in range(count):
                n = int(per_table[k][t])
                u = torch.rand(n, dtype=torch.float64, generator=self.g, device=self.dev)
                rank = (torch.searchsorted(cdf, u, right=True) if self.case["alpha"] > 0 else (u * r).long()).clamp_(max=r - 1)
                parts[k].append((rank * 15485863 + self.shift[t]) % r)
        zero = torch.zeros(1, dtype=torch.int64, device=self.dev)
        return [(torch.cat(p).contiguous(), torch.cat([zero, torch.cumsum(x.reshape(-1), 0)]).contiguous())
                for p, x in zip(parts, lens)]

    def gradient(self, B: int) -> torch.Tensor:
        """Gradient of the pooled embeddings, N(0, 1e-4^2)."""
        return torch.randn((B, self.case["T"], self.case["D"]), generator=self.g, device=self.dev) * 1e-4


def _buffers(case: dict, B: int, N: int, dev) -> dq.StepBuffers:
    b = dq.StepBuffers(case["T"], case["D"], B, N, dev)
    for name, v in vars(b).items():  # (entries past the number of unique rows are never written)
        if isinstance(v, torch.Tensor) and name != "workspace":
            v.zero_()
    return b


def _split(case: dict, indices: torch.Tensor, offsets: torch.Tensor, parts: int):
    """The batch cut into micro-batches of consecutive samples, each table-major again."""
    T, B = case["T"], case["B"]
    Bm = B // parts
    lens = torch.diff(offsets).reshape(T, B)
    bag_node = (torch.arange(B, device=offsets.device) // Bm).repeat(T)
    node = torch.repeat_interleave(bag_node, lens.reshape(-1))
    zero = torch.zeros(1, dtype=torch.int64, device=offsets.device)
    return [(indices[node == k].contiguous(),
             torch.cat([zero, torch.cumsum(lens[:, k * Bm:(k + 1) * Bm].reshape(-1), 0)]).contiguous()) for k in range(parts)]


class State:
    pass


def prepare(case: dict, seed: int) -> State:
    s = State()
    s.case, kind = case, case["kind"]
    d = Draws(case, seed)
    s.tables = d.tables()
    if kind == "refresh":
        # training has moved the weights since the last refresh
        s.tables.master.mul_(float(1.0 + 0.25 * torch.rand(1, generator=d.g, device=d.dev).item()))
        return s
    T, D, B = case["T"], case["D"], case["B"]
    s.mode = dq.FWD_PACKED if case["mode"] == "packed" else dq.FWD_MASTER
    s.bound = B * case["bag"]  # lookups of one table, at most: bags per table x the longest bag
    steps = case.get("steps", 1)
    s.batches = d.batches(steps, B)
    N = max(ix.numel() for ix, _ in s.batches)
    if kind == "serve":
        s.out = torch.zeros((B, T, D), dtype=torch.float32, device=d.dev)
        return s
    s.bufs = _buffers(case, B, N, d.dev)
    if kind in ("step", "ahead", "nodes"):
        s.grads = [d.gradient(B) for _ in range(steps)]
    if kind == "ahead":
        s.dd = [_buffers(case, B, N, d.dev) for _ in range(steps - 1)] + [s.bufs]
    if kind == "nodes":
        n = case["nodes"]
        s.parts = _split(case, *s.batches[0], n)
        Nm = T * (B // n) * case["bag"]  # lookups of a micro-batch, at most
        s.mb = [_buffers(case, B // n, Nm, d.dev) for _ in range(n)]
        s.cap = n * Nm
        s.m_rows = torch.zeros(s.cap, dtype=torch.int64, device=d.dev)
        s.m_tuo = torch.zeros(T + 1, dtype=torch.int32, device=d.dev)
        s.m_nu = torch.zeros(1, dtype=torch.int32, device=d.dev)
        s.m_sums = torch.zeros((s.cap, D), dtype=torch.int32, device=d.dev)
        s.m_ws = torch.empty(dq.dqrm_sparse_merge_workspace_bytes(T, D, n, s.cap), dtype=torch.uint8, device=d.dev)
    if kind == "train":
        _prepare_dense(s, d, seed)
    return s


def _prepare_dense(s: State, d: Draws, seed: int) -> None:
    case, B = s.case, s.case["B"]
    bot, top = mlp_dims(case)
    rng = np.random.default_rng(seed)
    layer = lambda i, o: ((rng.standard_normal((o, i)) * math.sqrt(2.0 / (i + o))).astype(np.float32),  # noqa: E731
                          (rng.standard_normal(o) * math.sqrt(1.0 / o)).astype(np.float32))
    bl = [layer(i, o) for i, o in zip(bot[:-1], bot[1:])]
    tl = [layer(i, o) for i, o in zip(top[:-1], top[1:])]
    s.model = dq.DenseModel(case["T"], case["D"], bot, [w for w, _ in bl], [b for _, b in bl], top, [w for w, _ in tl],
                            [b for _, b in tl], d.dev)
    s.x = torch.exp(torch.randn((B, bot[0]), generator=d.g, device=d.dev))
    s.y = (torch.rand(B, generator=d.g, device=d.dev) < 0.25).float()
    s.loss = torch.zeros(1, dtype=torch.float32, device=d.dev)
    s.grad_emb = torch.zeros((B, case["T"], case["D"]), dtype=torch.float32, device=d.dev)
    s.dense_ws = torch.empty(dq.dqrm_dense_workspace_bytes(s.model, B), dtype=torch.uint8, device=d.dev)
    s.quant, s.dense_out = None, []
    if case["wbits"] or case["gbits"]:
        P = dq.dqrm_dense_param_count(s.model)
        g = bool(case["gbits"])
        err = torch.zeros(P, dtype=torch.float32, device=d.dev) if g else None
        scale = torch.zeros(2 * (len(bl) + len(tl)), dtype=torch.float32, device=d.dev) if g else None
        codes = torch.zeros(P, dtype=torch.int8, device=d.dev) if g else None
        s.quant = dq.DenseQuant(weight_bits=case["wbits"], grad_bits=case["gbits"], grad_error=err, grad_scale=scale,
                                grad_codes=codes)
        s.dense_out = [t for t in (scale, codes) if t is not None]


# ---- one pass ---------------------------------------------------------------------------------------------------


def _dedupe_args(batch, b: dq.StepBuffers):
    return batch + (b.sorted_pos, b.uniq_rows, b.seg_offsets, b.table_uniq_offsets, b.num_unique, b.workspace)


def _rest(s: State, grad: torch.Tensor, N: int, dd: dq.StepBuffers, lr: float = LR) -> None:
    """Segment sums, INT8 codes and update, from the dedupe result in `dd`."""
    b = s.bufs
    dq.dqrm_segment_sum(s.tables, b.B, N, grad, b.values, None, dd.workspace)
    dq.dqrm_quant_update(s.tables, b.cap, N, b.values, dd.uniq_rows, dd.table_uniq_offsets, b.g_absmax, b.gq, b.g_scale, lr,
                         dd.workspace)


def _index_outputs(b: dq.StepBuffers):
    return [b.sorted_pos, b.uniq_rows, b.seg_offsets, b.table_uniq_offsets, b.num_unique]


def _step_outputs(s: State):
    b = s.bufs
    return _index_outputs(b) + [b.out, b.values, b.g_absmax, b.gq, b.g_scale, s.tables.master, s.tables.packed]


def run(s: State):
    case, kind = s.case, s.case["kind"]
    if kind == "refresh":
        dq.dqrm_find_scale(s.tables)
        dq.dqrm_pack_int4(s.tables)
        return [s.tables.w_scale, s.tables.packed]
    T, D, B = case["T"], case["D"], case["B"]
    indices, offsets = s.batches[0]
    if kind == "serve":
        dq.dqrm_embbag_fwd(s.tables, indices, offsets, B, s.mode, s.out)
        return s.out
    b = s.bufs
    if kind == "step":
        if case["calls"] == "five":
            dq.dqrm_fwd_bwd_step(s.tables, b, indices, offsets, s.grads[0], LR, s.mode)
        else:
            dq.dqrm_embbag_fwd(s.tables, indices, offsets, B, s.mode, b.out)
            dq.dqrm_dedupe_multi(s.tables, B, [_dedupe_args((indices, offsets), b)], max_table_lookups=s.bound)
            _rest(s, s.grads[0], indices.numel(), b)
        return _step_outputs(s)
    if kind == "ahead":
        dq.dqrm_dedupe_multi(s.tables, B, [_dedupe_args(batch, dd) for batch, dd in zip(s.batches, s.dd)],
                             max_table_lookups=s.bound)
        for (ix, off), dd, g in zip(s.batches, s.dd, s.grads):
            dq.dqrm_embbag_fwd(s.tables, ix, off, B, s.mode, b.out)
            _rest(s, g, ix.numel(), dd)
        return _step_outputs(s) + [t for dd in s.dd[:-1] for t in _index_outputs(dd)]
    if kind == "train":
        dq.dqrm_embbag_fwd(s.tables, indices, offsets, B, s.mode, b.out)
        dq.dqrm_dense_step_quant(s.model, s.quant, B, s.x, b.out, s.y, TRAIN_LR, s.loss, s.grad_emb, s.dense_ws)
        dq.dqrm_dedupe_multi(s.tables, B, [_dedupe_args((indices, offsets), b)], max_table_lookups=s.bound)
        _rest(s, s.grad_emb, indices.numel(), b, TRAIN_LR)
        m = s.model
        return _step_outputs(s) + [s.loss, s.grad_emb] + m.bot_w + m.bot_b + m.top_w + m.top_b + s.dense_out
    # nodes: forward of the whole batch, backward and codes of the micro-batches, one update
    n, mb = case["nodes"], s.mb
    Bm = B // n
    dq.dqrm_dedupe_multi(s.tables, Bm, [_dedupe_args(p, m) for p, m in zip(s.parts, mb)], max_table_lookups=Bm * case["bag"])
    dq.dqrm_embbag_fwd(s.tables, indices, offsets, B, s.mode, b.out)
    g = s.grads[0]
    dq.dqrm_segment_sum_multi(s.tables, Bm, [(s.parts[j][0].numel(), g[j * Bm:(j + 1) * Bm], m.values,
                                              m.g_absmax if j == 0 else None, m.workspace) for j, m in enumerate(mb)])
    dq.dqrm_grad_quant_int8_multi(T, D, [(m.values, m.table_uniq_offsets, mb[0].g_absmax, m.gq, m.g_scale) for m in mb])
    dq.dqrm_sparse_merge(s.tables, [(m.uniq_rows, m.table_uniq_offsets, m.gq) for m in mb], s.m_rows, s.m_tuo, s.m_nu,
                         s.m_sums, s.m_ws)
    dq.dqrm_sparse_update_sums(s.tables, s.cap, s.m_rows, s.m_tuo, s.m_sums, mb[0].g_scale, LR)
    return ([b.out, s.m_rows, s.m_tuo, s.m_nu, s.m_sums, mb[0].g_absmax, s.tables.master, s.tables.packed]
            + [t for m in mb for t in (m.uniq_rows, m.table_uniq_offsets, m.values, m.gq)])
