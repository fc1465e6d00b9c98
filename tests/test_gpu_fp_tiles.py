"""GPU: the FP32 / FP64 group-sum product at the edges of its work-groups.

Calls whose full tiles would leave CUs idle take quarter tiles; a split's sums
are the same chain of products either way, so T_b must be equal bit for bit, and
within rounding of the FP64 oracle's.
"""
import numpy as np
import pytest

from oracle import oracle as O

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("n, m, d", [(5, 7, 1000), (70, 58, 1024), (100, 300, 961)])
def test_quarter_and_full_tiles_agree(precision, n, m, d):
    g = np.random.default_rng(n)
    x = g.standard_normal((n + m, d)) + 0.5
    x = (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)
    X, Y = torch.from_numpy(x[:n].copy()).to(DEV), torch.from_numpy(x[n:].copy()).to(DEV)
    kw = dict(seed=6, precision=precision, want_T="f64")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    many = 256 * (cus // 16 + 1) + 3  # 16 column slots: at least one full tile per CU
    full = hbt.perm_test(X, Y, many, **kw)["T"]
    for B in (1, 63, 64, 65, 255, 256, 257, 1000):
        assert np.array_equal(hbt.perm_test(X, Y, B, **kw)["T"], full[:B]), B
    # the bars of test_gpu_parity.py: 1e-10 (FP64), 1e-5 (FP32) of |f(r1)| + |f(r2)|
    at = [0, 1, 255, 256, many - 1]
    ref = O.perm_stats_at(x[:n].astype(np.float64), x[n:].astype(np.float64), at, seed=6)
    scale = 2 * abs(np.log(d))
    assert np.all(np.abs(full[at] - ref["T"]) <= (1e-10 if precision == "f64" else 1e-5) * scale)
