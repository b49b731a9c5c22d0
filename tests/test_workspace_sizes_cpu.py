"""A workspace sized for the largest of a program's calls holds for its smaller ones."""
import pytest

from paper_2503_18402_amd import gsmi

pytestmark = pytest.mark.skipif(not gsmi.is_available(), reason="library not built")


def test_binning_workspace_does_not_depend_on_how_items_are_split_into_views():
    for views in (2, 3, 16, 32):
        for n in (1, 255, 257, 300, 513, 1025, 4097, 100_001):
            assert gsmi.gs_bin_sort_workspace_bytes(views, n, 1000) <= \
                gsmi.gs_bin_sort_workspace_bytes(1, views * n, 1000), (views, n)


def test_frequency_map_workspace_grows_with_the_image():
    size = gsmi.gs_frequency_map_workspace_bytes
    for a in (1, 67, 800, 4096):
        for b in range(1, 4096):
            assert size(a, b) <= size(a, b + 1), (a, b)
            assert size(b, a) <= size(b + 1, a), (b, a)
