"""GPU: the Householder fold of shared clouds at the edges of its kernels.

The coefficients go four rows to a wave (waves that cross from a pair to the
next), the splits' sums 256 rows to a work-group against tables of four
coefficients in segments of 512 (work-groups of several pairs, X sizes about
multiples of 4, 32 and 512).
"""
import numpy as np
import pytest

from paper_2605_08048_amd import synth

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from test_gpu_clouds import _check_against_oracle_and_batched, _cloud  # noqa: E402


@pytest.mark.parametrize("d, sizes, budgets", [
    (64, [2, 3, 4, 5, 6, 31, 33], [1, 2, 63, 64, 65, 100]),        # many pairs to a work-group
    (300, [127, 128, 129, 130, 511], [255, 256, 257, 40]),
    (768, [512, 513, 1030], [300, 213]),
    (1024, [1537, 30, 9], [129, 257]),
])
def test_fold_at_edges(d, sizes, budgets):
    g = np.random.default_rng(d)
    clouds = [_cloud(g, n, d, g.uniform(1.5, 3.0), synth.random_unit(g, d)) for n in sizes]
    k = len(sizes)
    px, py = np.divmod(np.arange(k * k), k)
    keep = px != py
    px, py = px[keep], py[keep]
    B = np.array([budgets[i % len(budgets)] for i in range(len(px))])
    _check_against_oracle_and_batched(clouds, px, py, B, seed=12)
