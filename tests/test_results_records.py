"""Result records from a byte tensor: its elements in order, whatever its strides,
in an array of its own."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_08048_amd import hbt  # noqa: E402

BYTES = torch.arange(6 * hbt.RESULT_BYTES).to(torch.uint8)


@pytest.mark.parametrize("t", [BYTES, BYTES.view(6, -1), BYTES[::2], BYTES.view(3, -1)[:, :hbt.RESULT_BYTES],
                               BYTES.view(-1, 6).t(), BYTES[1:1 + hbt.RESULT_BYTES], BYTES[:0]],
                         ids=["flat", "rows", "strided", "columns", "transposed", "offset", "empty"])
def test_records_are_the_tensors_bytes(t):
    r = hbt.results_to_numpy(t)
    assert r.tobytes() == t.numpy().tobytes() and r.dtype == hbt.RESULT_DTYPE and r.ndim == 1
    assert r.flags.writeable and not np.shares_memory(r, t.numpy())
