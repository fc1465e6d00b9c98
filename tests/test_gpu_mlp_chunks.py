"""GPU: the allocator network at the edges of its 64-row chunks (one row, a
chunk less and more one, more chunks than the gradient has work-groups).

Tolerances: forward as in test_gpu_allocator.py (n u times the magnitudes); the
gradient's per-row FP32 error signals are off by at most (12 + 64 + 64 + 64 + 8)
u relative to the magnitudes of their own terms, summed exactly in FP64.
"""
import numpy as np
import pytest

from oracle import budget as Bu

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import allocator as A  # noqa: E402
from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
U32 = 2.0 ** -24


def _case(rows):
    g = np.random.default_rng(rows)
    th = A.init_theta(g)
    th[28:] += g.normal(0, 0.05, th.size - 28)
    th = th.astype(np.float32).astype(np.float64)
    X = g.normal(0, 2, (rows, 12)).astype(np.float32).astype(np.float64)
    T = g.normal(0, 1, (rows, 2)).astype(np.float32).astype(np.float64)
    dev = [torch.as_tensor(a, dtype=torch.float32, device=DEV) for a in (th, X, T)]
    return th, X, T, dev


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 129, 64 * 512, 64 * 512 + 65])
def test_network_at_chunk_edges(rows):
    th, X, T, (dth, dX, dT) = _case(rows)
    P = Bu.unpack(np.abs(th))
    out, cache = Bu.mlp_forward(th, X)
    Xs, _, Z1, _, Z2 = [np.abs(a) for a in cache]
    mag = P["oshift"] + P["oscale"] * (((Xs @ P["W1"].T + P["b1"]) @ P["W2"].T + P["b2"]) @ P["W3"].T + P["b3"])
    got = hbt.mlp_forward(dX, dth).cpu().numpy()
    assert np.all(np.abs(got - out) <= 3 * 80 * U32 * mag)

    # scratch and outputs full of NaN: every word that is read was written
    hbt.workspace(hbt.lib().hbt_mlp_grad_workspace_size(rows), dX.device).fill_(255)
    grad = torch.full((hbt.MLP_PARAMS,), float("nan"), device=DEV)
    loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
    hbt.mlp_grad(dX, dT, dth, grad, loss)
    again, _ = hbt.mlp_grad(dX, dT, dth)
    assert torch.equal(grad[28:], again[28:])  # a fixed order
    grad = grad.cpu().numpy().astype(np.float64)
    assert np.isnan(grad[:28]).all()
    want = Bu.mlp_backward(th, cache, out, T)
    # the size of each parameter's terms (error signals bounded by their
    # magnitudes), for the rounding of one row's chain of products
    e = (mag + np.abs(T)) / P["oscale"] / rows
    d2 = e @ P["W3"]
    d1 = d2 @ P["W2"]
    size = np.concatenate([(d1.T @ Xs).ravel(), d1.sum(0), (d2.T @ Z1).ravel(), d2.sum(0), (e.T @ Z2).ravel(), e.sum(0)])
    # a unit within its rounding of 0 may sit on either side of the ReLU: its row's whole term
    A1, A2 = cache[1], cache[3]
    t1 = 16 * U32 * (Xs @ P["W1"].T + P["b1"])
    t2 = 80 * U32 * ((Xs @ P["W1"].T + P["b1"]) @ P["W2"].T + P["b2"])
    near = (np.abs(A1) <= t1).any(1) | (np.abs(A2) <= t2).any(1)
    flip = np.concatenate([(d1[near].T @ Xs[near]).ravel(), d1[near].sum(0), (d2[near].T @ Z1[near]).ravel(),
                           d2[near].sum(0), (e[near].T @ Z2[near]).ravel(), e[near].sum(0)])
    assert np.all(np.abs(grad[28:] - want[28:]) <= 220 * U32 * size + flip)
    ref = Bu.mlp_loss(th, out, T)
    assert abs(float(loss.item()) - ref) <= 2 * 240 * U32 * 0.5 * float(np.sum(((mag + np.abs(T)) / P["oscale"]) ** 2)) / rows
