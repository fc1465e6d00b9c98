"""GPU: hbt_align's column sums by phases of the X chunks (16-byte rows), at the
edges of chunks, phases and columns, and the test of every row in them.
"""
import numpy as np
import pytest

from oracle import oracle as O

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("d", [4, 252, 256, 260, 512, 772, 1024])
def test_sums_by_phase_and_row_test(d):
    g = np.random.default_rng(d)
    for n, m in [(2, 2), (3, 70), (5, 31), (127, 33), (128, 2), (129, 64), (131, 200), (640, 90)]:
        x = g.standard_normal((n + m, d)) + 0.3
        x = (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)
        X, Y = torch.from_numpy(x[:n].copy()).to(DEV), torch.from_numpy(x[n:].copy()).to(DEV)
        r = hbt.align(X, Y)
        want = O.align(x[:n].astype(np.float64), x[n:].astype(np.float64))
        assert r["status"] == want["status"] == 0
        # v is the difference of two means of unit rows over their lengths: n + m
        # additions, each within eps of a sum of at most n + m, so (n + m) eps over the
        # smaller length, four of them for both sums and both roundings of the lengths
        tol = 4 * (n + m) * 2.3e-16 / min(want["r_x"], want["r_y"])
        assert np.max(np.abs(r["v"].cpu().numpy() - want["v"])) <= tol, (n, m)
        # the store path of a test sums the same chunks: the same bits
        t = hbt.perm_test(X, Y, 10, precision="f32")
        assert t["t_obs"] == r["t_obs"] and t["r_x"] == r["r_x"] and t["r_y"] == r["r_y"], (n, m)
        # one row off unit length by 2e-4 anywhere in the pair is found
        for i in sorted({0, 1, n - 1, n // 2, n, n + m - 1}):
            z = x.copy()
            z[i] *= 1 + 2e-4
            bad = hbt.align(torch.from_numpy(z[:n].copy()).to(DEV), torch.from_numpy(z[n:].copy()).to(DEV))
            assert bad["status"] == hbt.ERR_NOT_UNIT, (n, m, i)
