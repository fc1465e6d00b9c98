"""GPU: batched calls whose tables the device builds, in every form of their
arguments (row offsets, split counts, Philox words, shared splits, both tile
widths, more pairs than one pass of the scans), against single-pair calls.

The same splits and rows give the same bits, so everything but the sums of T_b
over several blocks must be equal; a pair has one block here.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
FIELDS = ("count", "B", "n", "m", "n_recheck", "status", "t_obs", "t_mean", "t_sd", "p")


def _rows(g, n, d):
    x = g.standard_normal((n, d)) + 2.0
    return torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)


def _singles(Z, off, n, m, B, ids, check, **kw):
    for p in check:
        o, a, b = int(off[p]), int(n[p]), int(m[p])
        yield p, hbt.perm_test(Z[o:o + a].clone(), Z[o + a:o + a + b].clone(), int(B[p]), pair_index=int(ids[p]), **kw)


@pytest.mark.parametrize("precision", ["f32", "bf16x2", "i8x3", "bf16lazy"])
@pytest.mark.parametrize("form", ["plain", "offsets", "splits", "index", "all"])
def test_forms_of_a_batched_call(precision, form):
    g = np.random.default_rng(3)
    P = 23
    n, m = g.integers(2, 300, P), g.integers(2, 300, P)
    B, ids, kw = np.full(P, 40), np.arange(P, dtype=np.uint32), {}
    off = np.concatenate([[0], np.cumsum(n + m)])[:P]
    rows = int((n + m).sum())
    if form in ("offsets", "all"):  # pairs in another order, with gaps
        rows += 3 * P
        off = np.empty(P, dtype=np.int64)
        at = 3
        for p in g.permutation(P):
            off[p] = at
            at += n[p] + m[p] + int(g.integers(0, 3))
    if form in ("splits", "all"):
        B = g.integers(1, 1500, P)
        B[4], B[5] = 1024, 2048  # both tile widths
    if form in ("index", "all"):
        n[7:10], m[7:10], B[7:10] = n[7], m[7], B[7]
        off = np.concatenate([[0], np.cumsum(n + m)])[:P] if form == "index" else off
        if form == "all":  # rows of the resized pairs may overlap others'
            off[7:10] = 0
        rows = max(rows, int((off + n + m).max()))
        ids = g.integers(0, 2 ** 32, P).astype(np.uint32)
        ids[7:10] = ids[7]  # three pairs share their splits
        kw["pair_index"] = ids
    Z = _rows(g, rows, 64)
    r = hbt.perm_test_batched(Z, off, n, m, B, seed=5, precision=precision, **kw)
    for p, s in _singles(Z, off, n, m, B, ids, range(P), seed=5, precision=precision):
        for k in FIELDS:
            assert r[k][p] == s[k], (p, k)


@pytest.mark.parametrize("P", [511, 512, 513, 1300])
def test_more_pairs_than_one_pass_of_the_scans(P):
    g = np.random.default_rng(P)
    n, m = g.integers(2, 40, P), g.integers(2, 40, P)
    off = np.concatenate([[0], np.cumsum(n + m)])
    Z = _rows(g, int(off[-1]), 8)
    r = hbt.perm_test_batched(Z, off, n, m, np.full(P, 3), seed=1)
    assert np.all(r["status"] == 0) and np.array_equal(r["n"], n) and np.array_equal(r["m"], m)
    check = sorted({0, 1, 510, 511 % P, P // 2, P - 2, P - 1, min(512, P - 1), min(1024, P - 1)})
    for p, s in _singles(Z, off, n, m, np.full(P, 3), np.arange(P), check, seed=1, precision="bf16x2"):
        for k in FIELDS:
            assert r[k][p] == s[k], (p, k)


@pytest.mark.parametrize("gaps", [False, True])
@pytest.mark.parametrize("C, P", [(5, 17), (600, 520)])
def test_shared_clouds_equal_the_pairs_stored_apart(C, P, gaps):
    g = np.random.default_rng(C)
    rows = g.integers(2, 60 if C > 100 else 300, C)
    off = np.concatenate([[0], np.cumsum(rows + (2 if gaps else 0))])[:C] + (4 if gaps else 0)
    Z = _rows(g, int(off[-1] + rows[-1]), 64)
    px, py = g.integers(0, C, P), g.integers(0, C, P)
    B = g.integers(1, 60, P)
    ids = g.integers(0, 2 ** 32, P).astype(np.uint32) if gaps else None
    r = hbt.perm_test_clouds(Z, off, rows, px, py, B, seed=9, pair_index=ids)
    Za = torch.cat([Z[o:o + k] for x, y in zip(px, py) for o, k in ((off[x], rows[x]), (off[y], rows[y]))])
    n, m = rows[px], rows[py]
    s = hbt.perm_test_batched(Za, np.concatenate([[0], np.cumsum(n + m)]), n, m, B, seed=9, pair_index=ids)
    for k in ("count", "B", "n", "m", "status", "p"):
        assert np.array_equal(r[k], s[k]), k
    assert np.allclose(r["t_obs"], s["t_obs"], rtol=0, atol=1e-12 * (1 + np.abs(s["t_obs"]).max()))


@pytest.mark.parametrize("d", [64, 300, 700, 1024, 1100, 2500])
def test_alignment_does_not_depend_on_the_call(d):
    # one pair's column sums are added by many work-groups, a batch's by one per
    # pair; enough rows that every quarter of the chunks holds some
    g = np.random.default_rng(d)
    n, m = np.array([700, 20, 130] + [5] * 8), np.array([400, 900, 33] + [6] * 8)
    off = np.concatenate([[0], np.cumsum(n + m)])
    Z = _rows(g, int(off[-1]), d)
    r = hbt.perm_test_batched(Z, off, n, m, np.full(11, 30), seed=2)
    three = hbt.perm_test_batched(Z, off[:4], n[:3], m[:3], np.full(3, 30), seed=2)
    for p, s in _singles(Z, off, n, m, np.full(11, 30), np.arange(11), range(3), seed=2, precision="bf16x2"):
        for k in FIELDS + ("r_x", "r_y", "mu_cos", "tau"):
            assert r[k][p] == s[k] == three[k][p], (p, k)
