"""The back-transformation at the sizes where its kernels change shape, by the check and the
derived tolerances of the eigen-decomposition tests (eigenvalues and H of a weights step against
LAPACK's of the same Gram matrix, FP64).

Sizes 9 (a last group of one column), 66 and 194 (one reflector in the block after one and after
three full blocks of 64; a last group of two columns), 1150 (a size whose eight columns of Z
still fit a workgroup's LDS) and 1152 (the first beyond)."""
import pytest

from tests.gpu_util import say
from tests.test_gpu_eigh_sizes import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 32, 32, 3, 3, 1), (4, 32, 32, 6, 11, 1), (4, 32, 128, 2, 97, 1),
                                   (6, 64, 64, 10, 23, 5), (5, 64, 64, 16, 18, 4)])
def test_back_transformation(shape):
    say(f"back-transformation {shape} (s = {shape[3] * shape[4] * shape[5]})")
    check(shape)
