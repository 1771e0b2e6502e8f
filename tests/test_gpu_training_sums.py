"""The training network's sums: hidden inputs are fused multiply-adds over ascending inputs from the bias on.

Near zero the order of a sum decides the side of the ReLU, and one unit of one row on the other side moves the
gradient by more than all rounding.  The parameters here put every hidden unit's input within rounding of zero at
one of the rows, so that any other order gives another gradient.
"""
import numpy as np
import pytest

from oracle import learned as ol
from tests.helpers import gpu_available

D = 64   # distinct rows, one per hidden unit


def _chain(W, b, X):
    """float32 b_u + sum_i W_ui X_ri by fused multiply-adds over ascending i (products are exact in float64)."""
    z = np.broadcast_to(b.astype(np.float32), (len(X), len(b)))
    for i in range(W.shape[1]):
        z = (z.astype(np.float64) + np.outer(X[:, i], W[:, i])).astype(np.float32)
    return z.astype(np.float64)


def _bias_last(W, b, X):
    return (_chain(W, np.zeros_like(b), X) + b).astype(np.float32).astype(np.float64)


def _f32(v):
    return np.asarray(v, np.float32).astype(np.float64)


def _problem(seed):
    """Parameters and D rows; unit u of either hidden layer is within rounding of zero at row u."""
    rng = np.random.default_rng(seed)
    P = ol.init_params(seed)
    P["W3"] = _f32(rng.standard_normal(P["W3"].shape) * 0.1)
    P["b3"] = _f32(rng.standard_normal(4) * 0.1)
    rows = np.zeros((D, 12))
    rows[:, :7] = rng.uniform(-1.2, 1.2, (D, 7))
    Q = rng.choice([4, 8, 16], D)
    rows[:, 7:9] = rng.uniform(0, Q[:, None] - 1, (D, 2))
    rows[:, 9] = rng.uniform(0.5, 2.0, D)
    rows[:, 10] = Q
    rows = _f32(rows)
    X = rows[:, :7]
    P["b1"] = -_f32(np.einsum("ui,ui->u", P["W1"], X))
    a1 = np.maximum(_chain(P["W1"], P["b1"], X), 0.0)
    P["b2"] = -_f32(np.einsum("ui,ui->u", P["W2"], a1))
    return P, rows, a1


def _reference(P, rows, tgt):
    """Loss and gradient in float64, the hidden units on or off as the float32 chains have them."""
    X = rows[:, :7]
    z1 = _chain(P["W1"], P["b1"], X)
    z2 = _chain(P["W2"], P["b2"], np.maximum(z1, 0.0))
    on1, on2 = z1 > 0, z2 > 0
    a1 = (X @ P["W1"].T + P["b1"]) * on1
    a2 = (a1 @ P["W2"].T + P["b2"]) * on2
    out = a2 @ P["W3"].T + P["b3"]
    loss, d_out = 0.0, np.zeros_like(out)
    for p in range(2):
        ml, kl = rows[:, 7 + p] + out[:, p], rows[:, 9] * 2.0 ** out[:, 2 + p]
        assert np.abs(out[:, 2 + p]).max() < 3.9   # (the clamp's edge is another threshold)
        j = np.arange(16.0)
        d = j - ml[:, None]
        lg = np.where(j < rows[:, 10:11], -kl[:, None] * d * d, -np.inf)
        mx = lg.max(1)
        e = np.exp(lg - mx[:, None])
        Z = e.sum(1)
        dt = tgt[:, p] - ml
        loss += (kl * dt * dt + mx + np.log(Z)).mean()
        d_out[:, p] = -2 * kl * (tgt[:, p] - (e * j).sum(1) / Z)
        d_out[:, 2 + p] = (dt * dt - (e * d * d).sum(1) / Z) * kl * np.log(2.0)
    g = ol.mlp_backward(P, dict(a0=X, a1=a1, a2=a2, z1=np.where(on1, 1.0, -1.0), z2=np.where(on2, 1.0, -1.0)),
                        d_out / len(rows))
    return loss, ol.flatten(g)


def _case(seed, R):
    P, rows, _ = _problem(seed)
    pick = np.arange(R) % D
    rng = np.random.default_rng(seed + 100)
    rows = rows[pick]
    tgt = np.minimum(np.rint(np.abs(rows[:, 7:9] + rng.standard_normal((R, 2)))), rows[:, 10:11] - 1).astype(np.int64)
    return P, rows, tgt


def test_the_inputs_tell_the_orders_apart():
    P, rows, a1 = _problem(1)
    for W, b, X in ((P["W1"], P["b1"], rows[:, :7]), (P["W2"], P["b2"], a1)):
        z = _chain(W, b, X)
        scale = np.abs(W).sum(1) * np.abs(X).max()
        assert np.all(np.abs(np.diag(z)) < 64 * 2.0 ** -24 * scale)
        assert np.sum((z > 0) != (_bias_last(W, b, X) > 0)) >= 5


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("seed,R", [(1, 64), (2, 1000), (3, 4096), (4, 65536)])
def test_gradient_has_the_ordered_sums(seed, R):
    """2-norm within 1e-6: an entry passes four float32 sums of at most 64 terms (each about sqrt(64) 2^-25 of their
    size, 2.4e-7, 5e-7 together) and the sums over the rows, whose partial sums have no more terms than that."""
    import torch
    import paper_2407_06042_amd as dm
    P, rows, tgt = _case(seed, R)
    tr = dm.MlpTrainer(torch.from_numpy(ol.flatten(P).astype(np.float32)).cuda(), lr=1e-3)
    loss = float(tr.step(torch.from_numpy(rows.astype(np.float32)).cuda(),
                         torch.from_numpy(tgt.astype(np.int32)).cuda()).cpu().numpy()[0])
    lo, go = _reference(P, rows, tgt)
    assert abs(loss - lo) < 1e-6 * max(1.0, abs(lo))
    for got, scale in ((tr.grad, 1.0), (tr.m, 0.1)):
        g = got.cpu().numpy().astype(np.float64) / scale
        err = np.linalg.norm(g - go) / np.linalg.norm(go)
        print("rows %d: gradient error %.3g" % (R, err), flush=True)
        assert err < 1e-6


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_negative_precisions():
    """Rows whose logits grow away from the centre, by more than exp holds from the nearest level on.

    The exponents reach 4 2^0.5 16^2 = 1450, where float32 steps are 1.2e-4: the weights, and with them loss and
    gradient, within 1e-3."""
    import torch
    import paper_2407_06042_amd as dm
    P, rows, tgt = _case(7, 640)
    rows[:, 9] = -_f32(np.linspace(0.05, 4.0, len(rows)))
    tr = dm.MlpTrainer(torch.from_numpy(ol.flatten(P).astype(np.float32)).cuda(), lr=1e-3)
    loss = float(tr.step(torch.from_numpy(rows.astype(np.float32)).cuda(),
                         torch.from_numpy(tgt.astype(np.int32)).cuda()).cpu().numpy()[0])
    lo, go = _reference(P, rows, tgt)
    g = tr.grad.cpu().numpy().astype(np.float64)
    print("negative precisions: loss %.6g (%.6g), gradient error %.3g" % (loss, lo, np.linalg.norm(g - go) / np.linalg.norm(go)))
    assert abs(loss - lo) < 1e-3 * max(1.0, abs(lo))
    assert np.linalg.norm(g - go) < 1e-3 * np.linalg.norm(go)
