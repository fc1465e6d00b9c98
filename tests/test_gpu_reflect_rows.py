"""GPU: reflection and storage of rows that the 16-byte loads do not take, whole
rows in registers (d <= 1024 in FP32, 512 in FP64) and beyond, at the edges of
their columns, in every precision, against the FP64 oracle's statistics.
"""
import numpy as np
import pytest

from oracle import oracle as O

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
# per T_b, scaled by |f(r1)| + |f(r2)|: the bars of test_gpu_parity.py
TOL = {"f64": 1e-10, "f32": 1e-5, "bf16x2": 1e-4, "i8x3": 1e-4, "bf16e4m3": 1e-4}


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("dtype, d", [(np.float32, 61), (np.float32, 257), (np.float32, 511), (np.float32, 769),
                                      (np.float32, 1023), (np.float32, 1025), (np.float64, 256), (np.float64, 511),
                                      (np.float64, 513)])
def test_stored_rows_give_the_oracles_statistics(precision, dtype, d):
    g = np.random.default_rng(d)
    for n, m in [(3, 40), (33, 31), (95, 130)]:
        x = g.standard_normal((n + m, d)) + 0.4
        x = (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(dtype)
        X, Y = torch.from_numpy(x[:n].copy()).to(DEV), torch.from_numpy(x[n:].copy()).to(DEV)
        r = hbt.perm_test(X, Y, 300, seed=9, precision=precision, want_T="f64")
        assert r["status"] == 0
        at = O.perm_stats_at(x[:n].astype(np.float64), x[n:].astype(np.float64), np.arange(300), seed=9)
        f = lambda q: np.log(q * (d - q * q) / (1 - q * q))  # noqa: E731
        err = np.abs(r["T"] - at["T"]) / (np.abs(f(at["r1"])) + np.abs(f(at["r2"])))
        assert err.max() <= TOL[precision], (n, m, err.max())
