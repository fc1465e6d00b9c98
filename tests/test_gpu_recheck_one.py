"""GPU: one pair's recheck and end in one kernel, against the batched kernels.

Pairs of one and of several segments, with no flag to many: the counts, the number
of rechecked splits and the null moments (the rechecked T_b among them, summed in
one order) are the same bits as those of the pair in a batch of two.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt, synth  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("slots", [None, "0", "7"])
def test_one_pair_equals_the_pair_in_a_batch(slots, monkeypatch):
    if slots is not None:
        monkeypatch.setenv("HBT_RECHECK_SLOTS", slots)
    flagged = set()
    for k, (n, m, d, B) in enumerate([(20, 30, 64, 1), (20, 30, 64, 3000), (255, 257, 100, 900), (255, 257, 100, 9000),
                                      (256, 260, 1100, 2000), (2000, 900, 96, 500), (2000, 900, 96, 20000)] +
                                     [(30, 25, 64, B) for B in range(100, 1500, 100)] +
                                     [(400, 500, 96, B) for B in range(100, 1500, 100)]):
        g = np.random.default_rng(k)
        mu = synth.random_unit(g, d)
        rows = [synth.unit_rows(2.0 * mu + g.standard_normal((r, d)) / np.sqrt(d)).astype(np.float32) for r in (n, m)]
        X, Y = (torch.from_numpy(r).to(DEV) for r in rows)
        Z = torch.cat([X, Y, X, Y])
        for precision in ("bf16x2", "bf16lazy", "f32"):
            one = hbt.perm_test(X, Y, B, seed=5, precision=precision)
            if precision == "f32":
                assert one["status"] == 0 and 0 <= one["count"] <= B
                continue
            two = hbt.perm_test_batched(Z, [0, n + m], [n, n], [m, m], [B, 50], seed=5, precision=precision)[0]
            for f in ("status", "count", "p", "n_recheck", "t_obs", "t_mean", "t_sd"):
                assert one[f] == two[f], (n, m, B, precision, f, one[f], two[f])
            flagged.add(min(int(one["n_recheck"]), 2))
    assert flagged == {0, 1, 2}, flagged  # none, one and several
