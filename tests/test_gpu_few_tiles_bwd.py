"""The backward blend of launches that the list-parallel kernel takes, at the tile counts
where its shape changes."""
import pytest

from tests.few_tiles_util import step_kernel_us

pytestmark = pytest.mark.gpu


# 304 tiles of 16 against 256: 19% more work; a quarter is left for how the blocks fall on
# the CUs
@pytest.mark.parametrize("length", [10, 30, 100])
def test_more_tiles_than_wide_blocks_fit_do_not_queue(length):
    fits = step_kernel_us(256, 256, 16, length, "k_blend_bwd")
    more = step_kernel_us(304, 256, 16, length, "k_blend_bwd")
    assert more <= 1.5 * fits, (more, fits)
