"""GPU: the split stage's LDS limit of 64 KB a work-group, which one and two
work-groups per CU exceed: refused for pairs of every size, before any launch.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n,m", [(40, 50), (500, 600), (1500, 1400)])
def test_split_caps(n, m):
    g = np.random.default_rng(n)
    x = g.standard_normal((2 * (n + m), 64)) + 0.3
    Z = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)

    def calls():
        one = hbt.perm_test(Z[:n], Z[n:n + m], 300, seed=4, precision="bf16x2")
        two = hbt.perm_test_batched(Z, [0, n + m], [n, n], [m, m], 300, seed=4)
        return [tuple(one[f] for f in ("count", "t_mean", "t_sd")), tuple(two["count"]), tuple(two["t_mean"])]

    entry = hbt.tune_entry_get("bf16x2", 64)
    want = calls()
    try:
        hbt.tune_entry_set("bf16x2", 64, dict(entry, split_cap=3))
        assert calls() == want
        for cap in (1, 2):
            hbt.tune_entry_set("bf16x2", 64, dict(entry, split_cap=cap))
            with pytest.raises(hbt.HbtError) as e:
                hbt.perm_test(Z[:n], Z[n:n + m], 300, seed=4, precision="bf16x2")
            assert e.value.status == hbt.ERR_DEVICE
            with pytest.raises(hbt.HbtError) as e:
                hbt.perm_test_batched(Z, [0, n + m], [n, n], [m, m], 300, seed=4)
            assert e.value.status == hbt.ERR_DEVICE
    finally:
        hbt.tune_entry_set("bf16x2", 64, entry)
    assert calls() == want
