"""The list-parallel blends in the shapes they take from 513 tiles of 8 and 257 of 16 pixels
on, against the FP64 oracle: backward with 8 waves a tile, so that lists of more than eight
chunks (288 entries) give a wave several, and with the short lists in blocks of their own;
forward with four waves a tile, one chunk after the other at tiles of 16.  The images sit in
a view that is empty otherwise; tolerances as for the smaller views of the same lists (a
chunk of a list of 1025 entries has 65, so T is recovered over at most 65 divisions)."""
import pytest

from tests.test_gpu_blend_lists import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,w,h", [(8, 301, 201), (8, 397, 313), (16, 597, 395), (16, 797, 637)])
@pytest.mark.parametrize("count,kind", [(24, "plain"), (48, "clamped"), (49, "plain"), (300, "faint"),
                                        (385, "clamped"), (385, "dense"), (1025, "faint")])
def test_lists_of_more_tiles_match_oracle(tile, w, h, count, kind):
    _compare(w, h, tile, count, kind, least=0.5)
