"""GPU: the tables of a call of one pair, written by its first kernel.

Up to 2976 bytes go as an argument of the column sums (rows of 16-byte loads and
others); more splits need a longer tile list and a kernel of its own.  A split's
T_b does not depend on how many follow, so both must give the same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["f32", "f64", "bf16x2", "bf16lazy"])
@pytest.mark.parametrize("d", [61, 64, 1100])
def test_long_and_short_tables_agree(precision, d):
    g = np.random.default_rng(d)
    x = g.standard_normal((41, d)) + 0.4
    x = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)
    X, Y = x[:20].clone(), x[20:].clone()
    few = hbt.perm_test(X, Y, 300, seed=3, precision=precision, want_T="f64")
    many = hbt.perm_test(X, Y, 70000, seed=3, precision=precision, want_T="f64")
    assert few["status"] == many["status"] == 0 and few["t_obs"] == many["t_obs"]
    assert np.array_equal(few["T"], many["T"][:300])
    given = hbt.perm_test(X, Y, 300, precision=precision, want_T="f64",
                          masks=hbt.perm_test(X, Y, 300, seed=3, want_masks=True)["masks"])
    assert np.array_equal(given["T"], few["T"])
    a = hbt.align(X, Y)
    assert a["t_obs"] == few["t_obs"]
