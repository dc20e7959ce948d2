"""Dense total variation on both sides of the rule between its kernels, and at the walk's remainders (GPU)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_tv_walk import test_dense_tv as _check  # noqa: E402

pytestmark = pytest.mark.gpu


# 2^20 floats and planes of 256 float4 columns or more take the walk: x lengths that are no multiple of its run
# of four planes, columns that are no multiple of a block, the fewest planes, both sides of either limit
@pytest.mark.parametrize("shape", [(44, 44, 44, 12), (45, 45, 45, 12), (2, 210, 211, 12), (3, 173, 169, 12), (5, 97, 181, 12),
                                   (6, 150, 151, 8), (7, 129, 97, 12), (1025, 16, 16, 4), (1025, 15, 17, 4), (41, 41, 39, 16)])
def test_both_kernels(shape):
    _check(shape, 0.7)
