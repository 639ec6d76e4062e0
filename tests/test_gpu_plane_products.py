"""The precision that the dense part's products promise: operands as sums of three bfloat16, the six largest of their nine products.

A sum of K such products differs from float64 by some sqrt(K / 16) roundings of 2^-25 (K = 512: 1e-7 of the 2-norm, 2048: 2e-7).  Without
any one of the six products it is 2.4e-6 or more, whatever K is.  The gradients of a short model are a few products in a
row, 4e-7 together, so a bound of 1e-6 holds with all six and fails with five."""
import math

import numpy as np
import pytest

BOUND = 1e-6
SIX = [(p, s - p) for s in (2, 1, 0) for p in range(s + 1)]


def _bfloat16(x):
    u = x.view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _product(a, b, pairs):
    """a b^T by planes, added up as the matrix instructions do: 16 of the reduction at a time, two accumulators."""
    def planes(x):
        out = []
        for _ in range(3):
            out.append(_bfloat16(x))
            x = x - out[-1]
        return [p.astype(np.float64) for p in out]
    pa, pb = planes(a), planes(b)
    first = rest = np.zeros((len(a), len(b)), np.float32)
    for k in range(0, a.shape[1], 16):
        for p, q in pairs:
            t = pa[p][:, k:k + 16] @ pb[q][:, k:k + 16].T
            if p + q:
                rest = (rest + t).astype(np.float32)
            else:
                first = (first + t).astype(np.float32)
    return first + rest


@pytest.mark.parametrize("K", [20, 512, 2048])
def test_bound_tells_six_products_from_five(K):
    rng = np.random.default_rng(K)
    a, b = rng.standard_normal((128, K)).astype(np.float32), rng.standard_normal((64, K)).astype(np.float32)
    want = a.astype(np.float64) @ b.astype(np.float64).T
    error = lambda pairs: np.linalg.norm(_product(a, b, pairs) - want) / np.linalg.norm(want)  # noqa: E731
    assert error(SIX) < BOUND / 4
    assert all(error([x for x in SIX if x != left_out]) > 2 * BOUND for left_out in SIX)


def _margins(bot, top, x, emb):
    """How far a sample's pre-activations are from zero, at least, over their layer's root mean square."""
    T, D = emb.shape[1:]
    i, j = np.tril_indices(T + 1, -1)
    h, away = x.astype(np.float64), np.full(len(x), np.inf)
    for k, (w, b) in enumerate(bot + top[:-1]):
        if k == len(bot):
            Z = np.concatenate([h[:, None], emb], axis=1)
            h = np.concatenate([h, np.einsum("bpd,bpd->bp", Z[:, i], Z[:, j])], axis=1)
        z = h @ w.T.astype(np.float64) + b
        away, h = np.minimum(away, np.abs(z).min(axis=1) / np.sqrt((z * z).mean())), np.maximum(z, 0)
    return away


def _dims(layers):
    return [layers[0][0].shape[1]] + [w.shape[0] for w, _ in layers]


def _oracle_gradients(oracle, bot, top, x, emb, y):
    """The same from the float64 oracle."""
    f64 = lambda layers, k: [np.ascontiguousarray(layer[k], np.float64) for layer in layers]  # noqa: E731
    loss, grad, (bw, bb, tw, tb) = oracle.dense_step_ex(_dims(bot), f64(bot, 0), f64(bot, 1), _dims(top), f64(top, 0), f64(top, 1),
                                                        x, emb, y, 1.0, apply_sgd=False, want_grads=True)
    return loss, grad.reshape(emb.shape), list(zip(bw, bb)), list(zip(tw, tb))


def _layers(rng, dims):
    return [((rng.standard_normal((o, i)) * math.sqrt(2.0 / (i + o))).astype(np.float32), (rng.standard_normal(o) * 0.1).astype(np.float32))
            for i, o in zip(dims[:-1], dims[1:])]


def _gpu_gradients(T, D, bot, top, x, emb, y, bits=0):
    """The step's loss, gradient of emb, and per layer (dW, db): its FP32 gradients as the buffer of a group of micro-batches has them."""
    import torch
    import paper_2410_20046_amd as dq

    dev = torch.device("cuda:0")
    m = dq.DenseModel(T, D, _dims(bot), [w for w, _ in bot], [b for _, b in bot], _dims(top), [w for w, _ in top], [b for _, b in top], dev)
    flat = torch.zeros(dq.dqrm_dense_param_count(m), device=dev)
    ws = torch.empty(dq.dqrm_dense_workspace_bytes(m, len(x)), dtype=torch.uint8, device=dev)
    loss, grad = torch.zeros(1, device=dev), torch.zeros(emb.shape, device=dev)
    dq.dqrm_dense_step_quant(m, dq.DenseQuant(weight_bits=bits, grad_buffer=flat, buffer_add=False, buffer_update=False), len(x),
                             *(torch.from_numpy(a).to(dev) for a in (x, emb, y)), 1.0, loss, grad, ws)
    torch.cuda.synchronize()
    flat, out, at = flat.cpu().numpy(), [], 0
    for w, _ in top + bot:  # (the flat order)
        block = flat[at:at + w.shape[0] * (w.shape[1] + 1)].reshape(w.shape[0], -1)
        out.append((block[:, :-1], block[:, -1]))
        at += block.size
    return float(loss.item()), grad.cpu().numpy(), out[len(top):], out[:len(top)]


def _error(got, want):
    got = got.astype(np.float64)
    assert np.isfinite(got).all()
    return np.linalg.norm(got - want) / np.linalg.norm(want)


# Tiles (256 CUs): 64 x 64 at 700 samples; at 8190 128 x 128 for 512 columns, 128 x 64 for 256 and 250, each with its reduction along
# the rows of both operands (forward) and of one (input gradients).  Hidden layers of 3 to 5 outputs: reductions shorter than the 8
# floats that are read at a time.
@pytest.mark.gpu
@pytest.mark.parametrize("T,D,B,bot,top,seed", [
    (3, 16, 700, [20, 100], [130, 70], 1), (2, 16, 8190, [20, 256], [512, 250], 1), (2, 8, 65, [20, 5], [4, 3], 1),
    (2, 8, 1, [20, 5], [4, 3], 0)])
def test_gradients_to_the_precision_of_six_products(oracle, T, D, B, bot, top, seed):
    rng = np.random.default_rng(seed)
    bot, top = _layers(rng, bot + [D]), _layers(rng, [D + (T + 1) * T // 2] + top + [1])
    n = B + B // 10 + 20
    x, emb = rng.standard_normal((n, 20)).astype(np.float32), rng.standard_normal((n, T, D)).astype(np.float32)
    y = (rng.random(n) < 0.25).astype(np.float32)
    # samples without a pre-activation within 1e-5 of zero, where a ReLU's derivative depends on the rounding
    keep = np.flatnonzero(_margins(bot, top, x, emb) > 1e-5)[:B]
    x, emb, y = x[keep], emb[keep], y[keep]
    assert len(x) == B
    loss, demb, gbot, gtop = _oracle_gradients(oracle, bot, top, x, emb, y)
    got_loss, got_emb, got_bot, got_top = _gpu_gradients(T, D, bot, top, x, emb, y)
    assert abs(got_loss - loss) <= BOUND * abs(loss)
    errors = {"emb": _error(got_emb, demb)}
    for name, got, want in (("bot", got_bot, gbot), ("top", got_top, gtop)):
        for l, (g, w) in enumerate(zip(got, want)):
            errors[f"{name}_w[{l}]"], errors[f"{name}_b[{l}]"] = _error(g[0], w[0]), _error(g[1], w[1])
    print({k: float(f"{v:.2g}") for k, v in errors.items()}, flush=True)
    assert max(errors.values()) <= BOUND, errors


# A finite feature that rounds up to an infinite bfloat16, with weights so small that everything stays finite: its products are those of
# the floats.
@pytest.mark.gpu
@pytest.mark.parametrize("B", [70, 700, 8190])
def test_products_of_floats_next_to_the_largest(oracle, B):
    T, D, huge = 3, 32, np.float32(3.402e38)
    rng = np.random.default_rng(4)
    bot, top = _layers(rng, [20, 130, 140, D]), _layers(rng, [D + 6, 140, 129, 1])
    bot[0][0][:, 4] *= np.float32(1e-37)
    n = B + 50
    x, emb = rng.standard_normal((n, 20)).astype(np.float32), rng.standard_normal((n, T, D)).astype(np.float32)
    y = (rng.random(n) < 0.25).astype(np.float32)
    x[7, 4] = huge
    keep = np.flatnonzero(_margins(bot, top, x, emb) > 3e-6)[:B]
    x, emb, y = x[keep], emb[keep], y[keep]
    assert len(x) == B and (x == huge).sum() == 1
    loss, demb, gbot, gtop = _oracle_gradients(oracle, bot, top, x, emb, y)
    got_loss, got_emb, got_bot, got_top = _gpu_gradients(T, D, bot, top, x, emb, y)
    # (a few fp32 sums in a row, some 4e-7 of the 2-norm each.  By columns only the first layer, whose inputs are exact: of a hidden
    # unit that is hardly above zero a column has nothing but the rounding of that activation)
    assert abs(got_loss - loss) <= 1e-5 * abs(loss)
    assert _error(got_emb, demb) <= 1e-5
    assert max(_error(got_bot[0][0][:, c], gbot[0][0][:, c]) for c in range(20)) <= 1e-5
    for g, w in zip(got_bot[1:] + got_top, gbot[1:] + gtop):
        assert _error(g[0], w[0]) <= 1e-5 and _error(g[1], w[1]) <= 1e-5


# Quantised weights take three products, their codes as one plane (and, forward, the rounding of scale * code as another): the bound is
# that of six.  Tiles as above (at 8190 128 x 128, 128 x 64; at 700 64 x 64), reductions of less than a slab, of whole slabs and with a
# rest, inputs that fill a padded row and that do not; and layers so narrow, of so few samples, that not all codes find room (the others
# take six products).
@pytest.mark.gpu
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("T,D,B,bot,top,seed", [
    (3, 16, 700, [20, 100], [130, 70], 1), (2, 16, 8190, [20, 256], [512, 250], 1), (2, 8, 65, [64, 5], [4, 33], 1), (3, 64, 300, [128, 65], [97, 64], 2),
    (2, 8, 40, [20, 24, 17], [20], 3)])
def test_gradients_of_quantised_weights_to_the_same_precision(oracle, T, D, B, bot, top, seed, bits):
    rng = np.random.default_rng(seed)
    bot, top = _layers(rng, bot + [D]), _layers(rng, [D + (T + 1) * T // 2] + top + [1])
    used = lambda layers: [(oracle.mlp_fake_quant(w, bits)[0].reshape(w.shape), b) for w, b in layers]  # noqa: E731
    n = B + B // 10 + 20
    x, emb = rng.standard_normal((n, bot[0][0].shape[1])).astype(np.float32), rng.standard_normal((n, T, D)).astype(np.float32)
    y = (rng.random(n) < 0.25).astype(np.float32)
    keep = np.flatnonzero(_margins(used(bot), used(top), x, emb) > 1e-5)[:B]
    x, emb, y = x[keep], emb[keep], y[keep]
    assert len(x) == B
    loss, demb, gbot, gtop = _oracle_gradients(oracle, used(bot), used(top), x, emb, y)
    got_loss, got_emb, got_bot, got_top = _gpu_gradients(T, D, bot, top, x, emb, y, bits)
    assert abs(got_loss - loss) <= BOUND * abs(loss)
    errors = {"emb": _error(got_emb, demb)}
    for name, got, want in (("bot", got_bot, gbot), ("top", got_top, gtop)):
        for l, (g, w) in enumerate(zip(got, want)):
            errors[f"{name}_w[{l}]"], errors[f"{name}_b[{l}]"] = _error(g[0], w[0]), _error(g[1], w[1])
    print({k: float(f"{v:.2g}") for k, v in errors.items()}, flush=True)
    assert max(errors.values()) <= BOUND, errors
    # samples that are not finite: as with the same weights given as floats, and the others within the bound
    odd = np.array([0, B // 3, B // 2, B - 1])
    x[odd, 3] = np.inf, -np.inf, np.nan, 3.402e38
    _, with_odd, _, _ = _gpu_gradients(T, D, bot, top, x, emb, y, bits)
    _, as_floats, _, _ = _gpu_gradients(T, D, used(bot), used(top), x, emb, y)
    others = np.setdiff1d(np.arange(B), odd)
    assert _error(with_odd[others], demb[others]) <= BOUND  # (samples beside them are added up again too)
    assert np.array_equal(np.isnan(with_odd[odd]), np.isnan(as_floats[odd])) and np.array_equal(np.isinf(with_odd[odd]), np.isinf(as_floats[odd]))
    finite = np.isfinite(as_floats[odd])
    assert np.linalg.norm(with_odd[odd][finite] - as_floats[odd][finite]) <= 10 * BOUND * np.linalg.norm(as_floats[odd][finite])
