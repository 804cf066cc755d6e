"""The projections' plan (host only): which kernel a layer's sizes take."""
import pytest

from tests._util import gemm_plan


@pytest.mark.parametrize("Hq,rows", [(32768, 256), (65535, 256), (65536, 64), (131072, 64)])
@pytest.mark.parametrize("M,hidden", [(256, 1024), (1024, 16384)])
def test_tiles_stay_within_a_buffer_resource(M, hidden, Hq, rows):
    """A tile of 256 rows of K = 128 Hq values of X must span less than 2^32 bytes: the kernel's
    buffer resource holds no more, and reads past its range give zeros."""
    p = gemm_plan(M, hidden, 128 * Hq, False)
    assert p.rows == rows and min(p.rows, M) * 128 * Hq * 2 < 2 ** 32
