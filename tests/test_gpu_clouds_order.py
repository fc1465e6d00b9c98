"""GPU: shared clouds whose pairs lie below and above the four-row split kernel's
2048 padded items, in any order: the same launches, and the results of the same
pairs stored apart.
"""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
SIZES = [30, 45, 300, 260, 1500, 1400]
PAIRS = [(0, 1), (2, 3), (1, 2), (4, 5)]  # 256 to 2944 padded items, the last above
B = [300, 200, 100, 250]


def _clouds():
    g = np.random.default_rng(8)
    x = g.standard_normal((sum(SIZES), 64)) + 0.3
    Z = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)
    return Z, np.cumsum([0] + SIZES)[:-1]


def _call(order, **kw):
    Z, off = _clouds()
    p = [PAIRS[k] for k in order]
    return hbt.perm_test_clouds(Z, off, SIZES, [x for x, _ in p], [y for _, y in p], [B[k] for k in order], seed=2,
                                pair_index=order, **kw)


def _launches(order):
    """Nodes of the call's graph (it is captured, and never run)."""
    hip = hbt.lib()  # resolves the HIP runtime it is linked to as well
    hip.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    ws = torch.empty(1 << 26, dtype=torch.uint8, device=DEV)
    res = torch.empty(len(order) * hbt.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    Z, off = _clouds()
    p = [PAIRS[k] for k in order]
    graph, n = C.c_void_p(), C.c_size_t()
    assert hip.hipStreamBeginCapture(C.c_void_p(s.cuda_stream), 1) == 0  # thread-local
    try:
        hbt.perm_test_clouds(Z, off, SIZES, [x for x, _ in p], [y for _, y in p], [B[k] for k in order], seed=2,
                             pair_index=order, stream=s, sync=False, results=res, workspace=ws)
    finally:
        assert hip.hipStreamEndCapture(C.c_void_p(s.cuda_stream), C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    hip.hipGraphDestroy(graph)
    return n.value


@pytest.mark.parametrize("order", [[3, 0, 1, 2], [0, 3, 1, 2], [0, 1, 2, 3]])
def test_place_of_the_large_pair(order):
    first = _call([3, 0, 1, 2])
    got = _call(order)
    by_pair = lambda r, o, f: [r[f][o.index(k)] for k in range(4)]
    for f in ("count", "p", "n_recheck", "t_obs", "t_mean", "t_sd", "status"):
        assert by_pair(got, order, f) == by_pair(first, [3, 0, 1, 2], f), f
    Z, off = _clouds()
    apart = torch.cat([Z[off[c]:off[c] + SIZES[c]] for k in order for c in PAIRS[k]])
    n, m = [SIZES[PAIRS[k][0]] for k in order], [SIZES[PAIRS[k][1]] for k in order]
    rows = np.cumsum([0] + [a + b for a, b in zip(n, m)])[:-1]
    want = hbt.perm_test_batched(apart, rows, n, m, [B[k] for k in order], seed=2, pair_index=order)
    for f in ("count", "p", "status"):
        assert np.array_equal(got[f], want[f]), f
    assert _launches(order) == _launches([3, 0, 1, 2])
