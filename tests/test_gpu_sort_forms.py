"""Sorts of more than a million keys of capacity take 4 or 12 keys per thread by the live count: binning with 2^20
live pairs and instances (the line), one more, and far fewer, against numpy's lexicographic sort."""
import pytest

from test_gpu_binning_paths import test_binning_paths_match_lexsort as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,V,size,cap,visible,wide", [
    (1 << 20, 1, (640, 360), 1 << 21, 1.0, 1), ((1 << 20) + 1, 1, (640, 360), 1 << 21, 1.0, 1),
    ((1 << 20) + 1, 1, (640, 360), 1 << 24, 0.9, 1), (1_200_000, 1, (640, 360), (1 << 20) + 1, 0.001, 3),
    (1_100_000, 2, (640, 360), 3_000_001, 0.6, 2)])
def test_binning_by_live_count(n, V, size, cap, visible, wide):
    check(n, V, size, cap, visible, wide)
