"""GPU: split masks drawn four rows at a time, bit for bit against the oracle.

The four-row kernel takes pairs of up to 2048 padded items (rounds of 64
16-item blocks; up to 1024 with half the registers), larger pairs one row a
wave; rows of a wave may belong to several pairs and be fewer than four.
"""
import numpy as np
import pytest

from oracle import oracle as O

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
BIG = 1284168


def _rows(g, n, d):
    x = g.standard_normal((n, d)) + 2.0
    return torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)


@pytest.mark.parametrize("n, m", [(2, 2), (3, 13), (9, 8), (60, 68), (64, 65), (500, 524), (1000, 25), (30, 1122),
                                  (1020, 1028), (1024, 1025)])
@pytest.mark.parametrize("B, offset", [(1, 5), (7, 0), (22, 2 ** 32 - 22)])
def test_masks_of_partial_groups_of_rows(n, m, B, offset):
    g = np.random.default_rng(n + m)
    seed = 0x123456789abcdef0 + n
    r = hbt.perm_test(_rows(g, n, 8), _rows(g, m, 8), B, seed=seed, pair_index=3, perm_offset=offset, want_masks=True)
    want = np.stack([O.split_mask(seed, 3, offset + b, n + m, n) for b in range(B)])
    assert np.array_equal(r["masks"], want)


def test_masks_when_the_boundary_buckets_are_large():
    # splits BIG .. BIG + 3 of 2040 items have over 64 items between them in
    # their boundary buckets (found by drawing the keys of 10^6 splits)
    n, m = 1000, 1040
    P = [O.split_keys(0, 0, BIG + b, n + m)[0] for b in range(4)]
    assert sum(int(np.sum(p == np.sort(p)[n - 1])) for p in P) > 64
    g = np.random.default_rng(0)
    r = hbt.perm_test(_rows(g, n, 8), _rows(g, m, 8), 4, perm_offset=BIG, want_masks=True)
    assert np.array_equal(r["masks"], np.stack([O.split_mask(0, 0, BIG + b, n + m, n) for b in range(4)]))


def test_batch_of_small_and_large_pairs_equals_single_calls():
    g = np.random.default_rng(7)
    n = np.array([5, 700, 1500, 20, 1023, 40, 40, 3000, 9])
    m = np.array([7, 400, 900, 31, 1025, 30, 30, 1000, 120])
    B = np.array([13, 1, 3, 2, 17, 6, 6, 5, 257])
    ids = np.array([0, 1, 2, 3, 4, 5, 5, 7, 8], dtype=np.uint32)  # pairs 5 and 6 share their splits
    off = np.concatenate([[0], np.cumsum(n + m)])
    Z = _rows(g, int(off[-1]), 64)
    r = hbt.perm_test_batched(Z, off, n, m, B, seed=99, pair_index=ids)
    assert np.all(r["status"] == 0)
    for p in range(len(n)):
        o = int(off[p])
        s = hbt.perm_test(Z[o:o + n[p]], Z[o + n[p]:o + n[p] + m[p]], int(B[p]), seed=99, pair_index=int(ids[p]),
                          precision="bf16x2")
        for k in ("count", "n_recheck", "t_obs", "t_mean", "t_sd"):  # the same splits give the same bits
            assert r[k][p] == s[k], (p, k)
