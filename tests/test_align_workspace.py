"""Workspace of hbt_align: the column sums' phases (three more rows of sums per 128 X
rows) only for the row lengths that can take 16-byte loads.  (Sizes only: no GPU.)"""
import pytest

from paper_2605_08048_amd import hbt

pytestmark = pytest.mark.skipif(not hbt.LIB_PATH.exists(), reason="libhbt.so not built")


@pytest.mark.parametrize("n,m", [(2, 2), (129, 40), (60000, 3000)])
@pytest.mark.parametrize("d,phases", [(4, True), (1024, True), (1023, False), (301, False), (1028, False), (8192, False)])
def test_size(n, m, d, phases):
    x = -(-n // 128)
    rows = x + (-(-(n + m) // 128) * 128 // 32 - n // 32) + (3 * x if phases else 0)
    d_pad = -(-d // 64) * 64
    vectors = d_pad * (2 * 8 + 8 + 8 + 4)  # both sums, v, t in both types
    least = rows * (8 * d + 4) + vectors
    size = hbt.lib().hbt_align_workspace_size(n, m, d)
    assert least <= size <= least + 20 * 256 + 1024  # tables, records and alignment
