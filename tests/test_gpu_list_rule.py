"""The fixed-order sums on both sides of the rule between searched and sorted pairs, 2^23 look-ups
(reflections times tiles), with each fold on the searched side: the comparison, and its tolerance, of
test_gpu_list_reduce."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_list_reduce as L  # noqa: E402


# 49,962 reflections: 167 tiles are searched, 168 sorted
@pytest.mark.parametrize("width,height,tile_w,mirror", [(8, 1336, 0, 0), (168, 64, 0, 0), (64, 64, 16, 1), (64, 64, 16, 2),
                                                        (64, 64, 16, 3), (96, 96, 16, 3)])
def test_either_side_of_the_rule(width, height, tile_w, mirror):
    L.test_searched_against_sorted(width, height, tile_w, mirror)
