"""GPU: the column sums of rows that the 16-byte loads do not take (FP64 rows, d not
a multiple of 4, rows off a 16-byte boundary), at the edges of chunks, waves and
columns, and the test of every row in them.
"""
import numpy as np
import pytest

from oracle import oracle as O

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


def rows(g, k, d, dtype):
    x = g.standard_normal((k, d)) + 0.3
    return (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(dtype)


def off_by_one(x):
    """x on the device, its first value one element past a 16-byte boundary."""
    t = torch.empty(x.size + 1, dtype=torch.from_numpy(x).dtype, device=DEV)[1:].view(*x.shape)
    return t.copy_(torch.from_numpy(x))


@pytest.mark.parametrize("dtype, d", [(np.float32, 3), (np.float32, 255), (np.float32, 257), (np.float32, 513),
                                      (np.float32, 1023), (np.float32, 768), (np.float64, 64), (np.float64, 1024),
                                      (np.float32, 1025)])
def test_sums_and_row_test(dtype, d):
    g = np.random.default_rng(d)
    for n, m in [(2, 2), (8, 31), (9, 33), (127, 64), (129, 5), (260, 200)]:
        X, Y = rows(g, n, d, dtype), rows(g, m, d, dtype)
        r = hbt.align(off_by_one(X), off_by_one(Y))
        want = O.align(X.astype(np.float64), Y.astype(np.float64))
        # v is the difference of two means of unit rows over their lengths: n + m additions,
        # each within eps of a sum of at most n + m, so (n + m) eps over the smaller length,
        # four of them for both sums and both roundings of the lengths
        tol = 4 * (n + m) * 2.3e-16 / min(want["r_x"], want["r_y"])
        assert np.max(np.abs(r["v"].cpu().numpy() - want["v"])) <= tol, (n, m)
        # x - 2 (v . x) / (v . v) v: v's relative error four times, and the output's rounding
        tol = 4 * tol * np.sqrt(d) / np.sqrt(want["vv"]) + (6e-8 if dtype == np.float32 else d * 2.3e-16)
        assert np.max(np.abs(r["X_out"].cpu().numpy() - want["Xp"])) <= tol, (n, m)
        # one row off unit length by 2e-4 anywhere in the pair is found
        for i in sorted({0, n - 1, n // 2, n, n + m - 1, n + m // 2}):
            Z = np.concatenate([X, Y])
            Z[i] = Z[i] * (1 + 2e-4)
            bad = hbt.align(off_by_one(Z[:n].copy()), off_by_one(Z[n:].copy()))
            assert bad["status"] == hbt.ERR_NOT_UNIT, (n, m, i)
