"""GPU: the splits of a batched call in one stream with the alignment (up to 2^26
keys) and beside it: the pairs' results are the same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("clouds", [False, True])
def test_results_do_not_depend_on_the_stream_of_the_splits(clouds):
    g = np.random.default_rng(8)
    sizes = [30, 45, 300, 260, 1500, 1400]
    x = g.standard_normal((sum(sizes), 64)) + 0.3
    Z = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)
    off = np.cumsum([0] + sizes)[:-1]

    def run(pairs, last):
        B = [500] * (pairs - 1) + [last]
        if clouds:
            return hbt.perm_test_clouds(Z, off, sizes, [0, 2, 4][:pairs], [1, 3, 5][:pairs], B, seed=2)
        return hbt.perm_test_batched(Z, off[0::2][:pairs], sizes[0::2][:pairs], sizes[1::2][:pairs], B, seed=2)

    few = run(3, 500)      # 2 million keys
    many = run(3, 30000)   # 90 million: the last pair's
    again = run(2, 500)
    for f in ("count", "p", "n_recheck", "t_obs", "t_mean", "t_sd", "status"):
        assert np.array_equal(few[f][:2], many[f][:2]), f
        assert np.array_equal(few[f][:2], again[f]), f
