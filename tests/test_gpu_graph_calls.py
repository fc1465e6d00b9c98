"""GPU: captured calls replayed with other inputs in the same buffers and eager work
between the replays: every replay gives the bits of the eager call.

Pairs whose tables and counters the column sums write and clear (few splits), that
upload them and fork (more than 2^26 keys), in one block of splits and in several;
and a batch whose tile list goes up on a side stream.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2605_08048_amd import hbt  # noqa: E402

DEV = "cuda:0"
FIELDS = ("t_obs", "r_x", "r_y", "p", "t_mean", "t_sd", "count", "B", "n_recheck", "status")


def _rows(seed, n, d, dtype):
    g = np.random.default_rng(seed)
    mu = np.random.default_rng(0).standard_normal(d) / np.sqrt(d)  # clouds about one direction
    x = 1.5 * mu + g.standard_normal((n, d)) / np.sqrt(d)
    return torch.from_numpy(x / np.linalg.norm(x, axis=1, keepdims=True)).to(DEV, dtype)


def _replays(call, operands, fresh):
    """call() -> device tensors, captured and replayed on three sets of inputs."""
    hbt.workspace(1 << 28, torch.device(DEV))  # the cached one, no longer replaced below
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = call()
    for seed in range(3):
        for t, x in zip(operands, fresh(seed)):
            t.copy_(x)
        want = [t.clone() for t in call()]
        for t, x in zip(operands, fresh(seed + 50)):  # other eager work on the same workspace
            t.copy_(x)
        call()
        for t, x in zip(operands, fresh(seed)):
            t.copy_(x)
        for _ in range(2):
            for t in out:
                t.view(torch.uint8).fill_(0xff)
            g.replay()
            torch.cuda.synchronize()
            yield out, want


@pytest.mark.parametrize("n,m,d,B,precision,dtype,blocks",
                         [(50, 60, 64, 999, "f64", torch.float64, 0), (50, 60, 64, 999, "bf16x2", torch.float32, 0),
                          (777, 1333, 301, 3000, "bf16lazy", torch.float32, 0),
                          (2000, 1500, 64, 30000, "bf16x2", torch.float32, 0),
                          (300, 200, 64, 3000, "f32", torch.float32, 1000)])
def test_one_pair(n, m, d, B, precision, dtype, blocks):
    X, Y = _rows(1, n, d, dtype), _rows(2, m, d, dtype)

    def call():
        r = hbt.perm_test(X, Y, B, seed=3, precision=precision, block_perms=blocks, want_T="f64", want_masks=True,
                          sync=False)
        return [r["result"], r["T"], r["masks"]]

    for out, want in _replays(call, (X, Y), lambda s: (_rows(10 + s, n, d, dtype), _rows(30 + s, m, d, dtype))):
        a, b = hbt.results_to_numpy(out[0])[0], hbt.results_to_numpy(want[0])[0]
        assert all(a[f] == b[f] for f in FIELDS) and a["status"] == 0, (a, b)
        assert torch.equal(out[1], want[1]) and torch.equal(out[2], want[2])


@pytest.mark.parametrize("d", [64, 301])
def test_batch_with_a_long_tile_list(d):
    P, n, m, B = 40, 130, 140, 3000  # 480 tiles of 8 bytes, 1440 of 16: ten copies
    Z = _rows(1, P * (n + m), d, torch.float32)
    off = np.arange(P) * (n + m)
    call = lambda: [hbt.perm_test_batched(Z, off, [n] * P, [m] * P, B, seed=6, precision="f32", stat_route=1,
                                          sync=False)]
    for out, want in _replays(call, (Z,), lambda s: (_rows(10 + s, P * (n + m), d, torch.float32),)):
        a, b = hbt.results_to_numpy(out[0]), hbt.results_to_numpy(want[0])
        for f in FIELDS:
            assert np.array_equal(a[f], b[f]), f
        assert np.all(a["status"] == 0)
