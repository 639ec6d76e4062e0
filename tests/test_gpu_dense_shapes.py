"""The dense step's kernels at the edges of their tiles, against the float64 oracle: interactions of 2 .. 64 vectors of odd and
even widths, and layers whose widths and batch fall on, just below and just above the tiles of the products."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _model(rng, T, D, bot, top):
    V = T + 1
    bot, top = list(bot) + [D], [D + V * (V - 1) // 2] + list(top) + [1]
    layers = lambda dims: ([(rng.standard_normal((o, i)) * math.sqrt(2.0 / (i + o))).astype(np.float32)  # noqa: E731
                            for i, o in zip(dims[:-1], dims[1:])],
                           [(rng.standard_normal(o) * math.sqrt(1.0 / o)).astype(np.float32) for o in dims[1:]])
    return (bot, *layers(bot), top, *layers(top))


def _check(oracle, T, D, B, bot, top, seed=7, margin=False):
    import torch
    import paper_2410_20046_amd as dq

    print(f"T={T} D={D} B={B} bot={bot} top={top}", flush=True)
    rng = np.random.default_rng(seed)
    bot_dims, bw, bb, top_dims, tw, tb = _model(rng, T, D, bot, top)
    x = np.exp(rng.standard_normal((B, bot_dims[0]))).astype(np.float32)
    if margin:  # biases of +-1 and sums of some 0.05: no pre-activation near zero, half of the units on
        x = rng.uniform(0.5, 2.0, x.shape).astype(np.float32)
        bw, tw = [w * np.float32(0.02) for w in bw], [w * np.float32(0.02) for w in tw]
        bb, tb = [np.sign(b) for b in bb], [np.sign(b) for b in tb]
    y = (rng.random(B) < 0.25).astype(np.float32)
    emb = (rng.standard_normal((B, T, D)) * 0.25).astype(np.float32)
    dev = torch.device("cuda:0")
    m = dq.DenseModel(T, D, bot_dims, bw, bb, top_dims, tw, tb, dev)
    ws = torch.empty(dq.dqrm_dense_workspace_bytes(m, B), dtype=torch.uint8, device=dev)
    loss = torch.zeros(1, dtype=torch.float32, device=dev)
    # both start 4 bytes past a 16-byte boundary
    buf = torch.zeros(2 * (B * T * D + 8), dtype=torch.float32, device=dev)
    n = B * T * D
    emb_d, grad = buf[1:1 + n].view(B, T, D), buf[(n + 8) // 4 * 4 + 1:][:n].view(B, T, D)
    emb_d.copy_(torch.from_numpy(emb))
    dq.dqrm_dense_step(m, B, torch.from_numpy(x).to(dev), emb_d, torch.from_numpy(y).to(dev), 1.0, loss, grad, ws)
    torch.cuda.synchronize()
    f64 = lambda l: [np.ascontiguousarray(a, np.float64) for a in l]  # noqa: E731
    BW, BB, TW, TB = f64(bw), f64(bb), f64(tw), f64(tb)
    loss_o, grad_o = oracle.dense_step(bot_dims, BW, BB, top_dims, TW, TB, x, emb, y, 1.0)
    assert abs(float(loss.item()) - loss_o) <= 1e-5 * max(1.0, abs(loss_o))
    # Up to 8 products in a row, each a sum of at most ~2000 terms with a relative error of about sqrt(2000) * 2^-24 =
    # 2.7e-6: 2e-5 of the 2-norm.  A pre-activation within that of zero may flip its ReLU's derivative: five times that.
    close = lambda got, exp, what: (np.linalg.norm(got.astype(np.float64) - exp) <= 1e-4 * np.linalg.norm(exp)) or pytest.fail(  # noqa: E731
        f"{what}: {np.linalg.norm(got.astype(np.float64) - exp) / np.linalg.norm(exp):.3g}")
    close(grad.cpu().numpy(), grad_o.reshape(B, T, D), "grad_emb")
    for name, got, before, exp in (("bot_w", m.bot_w, bw, BW), ("bot_b", m.bot_b, bb, BB), ("top_w", m.top_w, tw, TW), ("top_b", m.top_b, tb, TB)):
        for l, (g, w, e) in enumerate(zip(got, before, exp)):
            # the step itself (learning rate 1): the rounding of the weights is one part in 2^24 of them
            step, want = g.cpu().numpy().astype(np.float64) - w, e - w
            slack = 2.0 ** -24 * np.linalg.norm(w)
            err = np.linalg.norm(step - want)
            assert err <= 1e-4 * np.linalg.norm(want) + 2 * slack, (name, l, err, np.linalg.norm(want), slack)


@pytest.mark.parametrize("T,D,B,bot", [
    (1, 1, 3, [4]), (1, 16, 5, [13, 20]), (30, 12, 9, [13, 24]), (31, 20, 21, [13, 32]), (32, 8, 33, [9, 8]), (33, 24, 18, [13, 300]),
    (63, 64, 70, [13, 64]), (40, 7, 37, [5, 11]), (2, 130, 40, [13, 16]), (1, 1500, 6, [3]), (26, 64, 130, [13, 512, 256]),
    (5, 33, 64, [17, 120]), (15, 256, 24, [7, 8]), (26, 16, 40, [13, 280]), (26, 16, 41, [13, 288]),
    # both sides of the line between the plain kernels and the matrix cores, with and without the last layer riding along
    (31, 21, 19, [13, 64]), (62, 33, 10, [13, 48]), (20, 16, 30, [13, 64]), (21, 16, 30, [13, 64]), (15, 32, 31, [13, 256]),
    (14, 32, 31, [13, 256]), (14, 32, 31, [13, 300]), (26, 8, 130, [13, 64]), (33, 32, 9, [13, 600]), (50, 16, 9, [13, 64]), (48, 16, 33, [13, 64])])
def test_interaction_shapes(oracle, T, D, B, bot):
    _check(oracle, T, D, B, bot, [16])


# The products' tiles: layers just below, at and above one and two tiles of 64, batches of one sample, one partial
# slab and many slices.  Among the 2 million pre-activations of
# such a batch about 2e6 * 2.7e-6 * 0.8 = 4 lie within their rounding of zero, and each ReLU so flipped moves the embedding
# gradients by some 1e-3 of their norm; large batches therefore keep every pre-activation away from zero.
@pytest.mark.parametrize("T,D,B,bot,top", [
    (3, 64, 65, [13, 64, 64], [64, 65]), (2, 8, 1, [64, 128], [64, 64]), (3, 70, 129, [65, 64, 128], [63, 64, 127, 128]),
    (2, 8, 2085, [13, 300], [321, 257]), (2, 16, 8200, [16], [120, 260]), (2, 16, 4160, [64], [160, 256, 64]),
    (8, 16, 1023, [13, 48, 32], [60, 48]), (8, 64, 1536, [13, 64], [128, 64]), (3, 16, 257, [13, 600], [601, 64])])
def test_product_tiles(oracle, T, D, B, bot, top):
    _check(oracle, T, D, B, bot, top, margin=B > 1000)


# The products by planes of bfloat16: reductions below, at and above 8 (the shortest), a slab of 32 or 64 and two of them; columns and
# samples that end inside a tile of each size (128 x 128 and 128 x 64 from some 4096 samples on).
@pytest.mark.parametrize("T,D,B,bot,top", [
    (2, 16, 70, [7, 33], [9, 8]), (2, 16, 7, [8, 65], [31, 33]), (2, 8, 63, [9, 127], [63, 32]), (1, 62, 64, [20, 129], [65, 95]),
    (1, 64, 127, [17, 191], [96, 128]), (3, 60, 300, [18, 401], [384, 70]), (2, 16, 4097, [20, 190], [257, 70]),
    (2, 16, 8193, [8, 129], [385, 130])])
def test_plane_products(oracle, T, D, B, bot, top):
    _check(oracle, T, D, B, bot, top, margin=B > 1000)


# The last, smaller batch of an epoch in the workspace of the others: more slices of its weight gradients than of theirs.
def test_smaller_batch_in_the_workspace_of_a_larger():
    import torch
    import paper_2410_20046_amd as dq

    T, D, B = 25, 16, 4026
    rng = np.random.default_rng(2)
    dev = torch.device("cuda:0")
    model = _model(rng, T, D, [7, 172, 52, 420], [256])
    x, emb, y = (torch.from_numpy(a.astype(np.float32)).to(dev) for a in (
        rng.standard_normal((B, 7)), rng.standard_normal((B, T, D)) * 0.25, rng.random(B) < 0.25))
    results = []
    for sized_for in (B, 4096):
        m = dq.DenseModel(T, D, *model[:3], *model[3:], dev)
        size = dq.dqrm_dense_workspace_bytes(m, sized_for)
        room = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=dev)
        loss, grad = torch.zeros(1, device=dev), torch.zeros((B, T, D), device=dev)
        dq.dqrm_dense_step(m, B, x, emb, y, 1.0, loss, grad, room[:size])
        assert bool((room[size:] == 0xFF).all())
        results.append([t.cpu().numpy().view(np.uint32) for t in [loss, grad] + m.bot_w + m.bot_b + m.top_w + m.top_b])
    assert all(np.array_equal(a, b) for a, b in zip(*results))


# An infinite feature, as the floats' products have it: the first layer's outputs are infinite where its weight is positive (else 0
# after the ReLU), so the weight gradients of that feature's column and of those outputs' columns are not finite.  The second layer
# adds up infinities of both signs: NaN, which its ReLU makes 0.  Everything else is finite.
@pytest.mark.parametrize("B", [70, 700, 8200])
def test_products_of_infinities(B):
    import torch
    import paper_2410_20046_amd as dq

    T, D = 3, 32
    rng = np.random.default_rng(3)
    bot_dims, bw, bb, top_dims, tw, tb = _model(rng, T, D, [13, 130, 140], [140, 129])
    x, emb = rng.standard_normal((B, 13)).astype(np.float32), rng.standard_normal((B, T, D)).astype(np.float32)
    y = (rng.random(B) < 0.25).astype(np.float32)
    x[B // 2, 4] = np.inf
    dev = torch.device("cuda:0")
    m = dq.DenseModel(T, D, bot_dims, bw, bb, top_dims, tw, tb, dev)
    ws = torch.zeros(dq.dqrm_dense_workspace_bytes(m, B), dtype=torch.uint8, device=dev)
    loss, grad = torch.zeros(1, device=dev), torch.zeros((B, T, D), device=dev)
    dq.dqrm_dense_step(m, B, torch.from_numpy(x).to(dev), torch.from_numpy(emb).to(dev), torch.from_numpy(y).to(dev), 1.0, loss, grad, ws)
    finite = [torch.isfinite(t).cpu().numpy() for t in m.bot_w]
    assert np.array_equal(finite[0], np.broadcast_to(np.arange(13) != 4, (130, 13)))
    assert np.array_equal(finite[1], np.broadcast_to(bw[0][:, 4] < 0, (140, 130)))
    assert finite[2].all() and all(bool(torch.isfinite(t).all()) for t in [loss, grad] + m.bot_b + m.top_w + m.top_b)


# The short-input layer takes 4 samples to a workgroup while that fills 2 workgroups per CU or the layer has at most 256 outputs,
# then up to 16: remainders of 8, 16 and 16 samples (on 256 CUs).
@pytest.mark.parametrize("B", [4099, 8195, 9001])
@pytest.mark.parametrize("width", [68, 256, 260])
def test_short_input_layer(oracle, B, width):
    _check(oracle, 2, 8, B, [13, width], [16], margin=True)
