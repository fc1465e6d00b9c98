"""GPU: one pair's recheck and end in one kernel, against the batched kernels, for
the FP32 product and for FP64 input rows (half as many rows in flight): pairs of one
and of several segments, with no flag, one and many.  The same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt, synth  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision,dtype", [("f32", np.float32), ("f32", np.float64), ("bf16x2", np.float64)])
@pytest.mark.parametrize("slots", [None, "0", "7"])
def test_one_pair_equals_the_pair_in_a_batch(precision, dtype, slots, monkeypatch):
    if slots is not None:
        monkeypatch.setenv("HBT_RECHECK_SLOTS", slots)
    flagged = set()
    # (clouds of 3 and 4 rows have 35 splits, each drawn many times: those equal
    # to the observed one are flagged)
    for k, (n, m, d, B) in enumerate([(3, 4, 64, 1), (3, 4, 64, 400), (20, 30, 64, 3000), (256, 260, 1100, 2000),
                                      (2000, 900, 96, 20000), (2, 700, 64, 5000)] +
                                     [(3, 4, 64, B) for B in range(10, 100, 10)] +
                                     [(400, 500, 96, B) for B in range(1000, 8000, 1000)]):
        g = np.random.default_rng(k)
        mu = synth.random_unit(g, d)
        rows = [synth.unit_rows(2.0 * mu + g.standard_normal((r, d)) / np.sqrt(d)).astype(dtype) for r in (n, m)]
        X, Y = (torch.from_numpy(r).to(DEV) for r in rows)
        one = hbt.perm_test(X, Y, B, seed=5, precision=precision)
        two = hbt.perm_test_batched(torch.cat([X, Y, X, Y]), [0, n + m], [n, n], [m, m], [B, 50], seed=5,
                                    precision=precision)[0]
        for f in ("status", "count", "p", "n_recheck", "t_obs", "t_mean", "t_sd"):
            assert one[f] == two[f], (n, m, B, f, one[f], two[f])
        flagged.add((n + m > 512, min(int(one["n_recheck"]), 2)))
    assert {c for _, c in flagged} == {0, 1, 2} and (True, 2) in flagged, flagged
