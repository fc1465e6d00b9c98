"""GPU: the allocator network of many rows (one thread per row above 14 chunks of 64
rows per CU) gives the bits of the same rows in small calls.
"""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import numpy as np  # noqa: E402

from paper_2605_08048_amd import allocator as A  # noqa: E402
from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
PIECE = 8192


@pytest.mark.parametrize("extra", [0, 1, 257, 300001])
def test_rows_do_not_depend_on_the_call(extra):
    rows = 14 * 64 * torch.cuda.get_device_properties(0).multi_processor_count + extra
    g = np.random.default_rng(3)
    th = A.init_theta(g)
    th[28:] += g.normal(0, 0.05, th.size - 28)
    th = torch.as_tensor(th, dtype=torch.float32, device=DEV)
    X = torch.as_tensor(g.normal(0, 2, (rows, 12)), dtype=torch.float32, device=DEV)
    X[5, 3] = float("nan")  # its units of layer 1 become 0, as in the small call
    X[rows - 1, 7] = float("inf")
    whole = hbt.mlp_forward(X, th)
    parts = torch.cat([hbt.mlp_forward(X[k:k + PIECE], th) for k in range(0, rows, PIECE)])
    assert torch.equal(whole.view(torch.int32), parts.view(torch.int32))


class _KernelNode(C.Structure):  # hipKernelNodeParams
    _fields_ = [("block", C.c_uint * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint * 3),
                ("params", C.c_void_p), ("lds", C.c_uint)]


def test_launch():
    """The launch itself, from a captured call (never run): 179 us a million rows in
    chunks of 64, 161 with a thread per row."""
    hip = hbt.lib()  # resolves the HIP runtime it is linked to as well
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    th = torch.zeros(hbt.MLP_PARAMS, device=DEV)
    for rows, threads, per_group in [(14 * 64 * cus, 512, 64), (14 * 64 * cus + 1, 256, 256)]:
        X, out = torch.zeros(rows, 12, device=DEV), torch.zeros(rows, 2, device=DEV)
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph, node, n = C.c_void_p(), C.c_void_p(), C.c_size_t(1)
        assert hip.hipStreamBeginCapture(C.c_void_p(s.cuda_stream), 1) == 0  # thread-local
        status = hip.hbt_mlp_forward(rows, C.c_void_p(X.data_ptr()), C.c_void_p(th.data_ptr()),
                                     C.c_void_p(out.data_ptr()), C.c_void_p(s.cuda_stream))
        assert hip.hipStreamEndCapture(C.c_void_p(s.cuda_stream), C.byref(graph)) == 0 and status == hbt.OK
        assert hip.hipGraphGetNodes(graph, C.byref(node), C.byref(n)) == 0 and n.value == 1
        k = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(node, C.byref(k)) == 0
        hip.hipGraphDestroy(graph)
        assert (k.block[0], k.grid[0]) == (threads, -(-rows // per_group))
