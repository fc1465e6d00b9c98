"""GPU: tile lists of a few copies (on the caller's stream) and of many (on a side
stream): neither the splits nor the alignment wait for them, and the pairs' results
are those of single calls.
"""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"


def _batch(P, n, m, d):
    g = np.random.default_rng(P)
    x = g.standard_normal((P * (n + m), d)) + 0.3
    Z = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)).to(DEV)
    return Z, np.arange(P) * (n + m)


class _KernelNode(C.Structure):  # hipKernelNodeParams
    _fields_ = [("block", C.c_uint * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint * 3),
                ("params", C.c_void_p), ("lds", C.c_uint)]


def _copies_ahead(call):
    """Of each kernel of a captured call (never run): the k_upload launches it waits for."""
    hip = hbt.lib()  # resolves the HIP runtime it is linked to as well
    hip.hipKernelNameRefByPtr.restype = C.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [C.c_void_p, C.c_void_p]
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = C.c_void_p()
    assert hip.hipStreamBeginCapture(C.c_void_p(s.cuda_stream), 1) == 0  # thread-local
    try:
        call(s)
    finally:
        assert hip.hipStreamEndCapture(C.c_void_p(s.cuda_stream), C.byref(graph)) == 0
    n = C.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    e = C.c_size_t()
    assert hip.hipGraphGetEdges(graph, None, None, C.byref(e)) == 0
    a, b = (C.c_void_p * e.value)(), (C.c_void_p * e.value)()
    assert hip.hipGraphGetEdges(graph, a, b, C.byref(e)) == 0
    name, before = {}, {v: set() for v in nodes}
    for v in nodes:
        kind, k = C.c_int(), _KernelNode()
        assert hip.hipGraphNodeGetType(C.c_void_p(v), C.byref(kind)) == 0
        if kind.value == 0:
            assert hip.hipGraphKernelNodeGetParams(C.c_void_p(v), C.byref(k)) == 0
            name[v] = hip.hipKernelNameRefByPtr(k.func, None).decode()
    into = {v: [x for x, y in zip(a, b) if y == v] for v in nodes}
    done = []
    while len(done) < n.value:
        for v in nodes:
            if v not in done and all(u in done for u in into[v]):
                before[v] = set().union(*([before[u] | {u} for u in into[v]] or [set()]))
                done.append(v)
    hip.hipGraphDestroy(graph)
    return [(name[v], sum("k_upload" in name.get(u, "") for u in before[v])) for v in nodes if v in name]


@pytest.mark.parametrize("precision,route", [("f32", 0), ("f64", 0), ("f32", 1), ("bf16x2", 1)])
@pytest.mark.parametrize("P,B", [(6, 300), (40, 3000), (40, 30000)])
def test_lists(precision, route, P, B):
    n, m, d = 130, 140, 64
    Z, off = _batch(P, n, m, d)
    kw = dict(seed=6, precision=precision, stat_route=route)
    got = hbt.perm_test_batched(Z, off, [n] * P, [m] * P, B, **kw)
    for p in (0, P - 1):
        X = Z[off[p]:off[p] + n + m]
        one = hbt.perm_test(X[:n], X[n:], B, pair_index=p, **kw)
        for f in ("status", "count", "p", "t_obs", "n_recheck"):
            assert got[f][p] == one[f], f
    again = hbt.perm_test_batched(Z, off, [n] * P, [m] * P, B, **kw)
    assert np.array_equal(got, again)

    need = hbt.batched_workspace_size(off, [n] * P, [m] * P, B, d, precision=precision, stat_route=route)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    res = torch.empty(P * hbt.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    ahead = _copies_ahead(lambda s: hbt.perm_test_batched(Z, off, [n] * P, [m] * P, B, stream=s, sync=False,
                                                          results=res, workspace=ws, **kw))
    total = sum("k_upload" in k for k, _ in ahead)
    tiles = P * -(-B // 256)  # 8 bytes each, and 16 for each 128 of the 384 padded rows
    assert total >= 1 + (tiles * (8 if precision != "bf16x2" else 0) + tiles * 48 * route) // 3072
    for k, c in ahead:
        if any(x in k for x in ("k_split", "k_colsum", "k_finalize", "k_reflect")):
            assert c == 1, (k, c)  # the description that the tables are built from
