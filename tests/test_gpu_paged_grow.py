"""The one-launch append over small layers: both workgroup sizes and both ways of granting pages, at the numbers of segments
where they change (64 segments, 8 KB of new K rows).  Bit for bit against the model of the layout."""
import pytest

import test_gpu_paged

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B,H", [(128, 31, 1), (128, 16, 2), (128, 33, 1), (128, 32, 2), (128, 65, 1), (64, 63, 1),
                                   (64, 32, 2), (64, 65, 1), (64, 7, 1)])
def test_append_of_small_layers(D, B, H):
    test_gpu_paged.test_append_on_both_sides_of_the_one_launch_limit(D, B, H)
