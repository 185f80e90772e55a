"""The deferred-epilogue GEMM: the residual under contractions of as few stages as it takes."""
import pytest

from gpu_util import PEN
from test_gpu_fp8_linear import test_fwd_residual_on_the_deferred_kernels as check_residual

pytestmark = pytest.mark.gpu


# five stages of write-out, five of the residual and the last one (11 in all), one more; one tile and a second one
@pytest.mark.parametrize("case", [(15, 256, 1408, 256, PEN), (15, 512, 1408, 512, None), (15, 8448, 1408, 2048, PEN),
                                  (15, 8448, 1536, 2048, None)])
def test_residual_under_short_contractions(case):
    check_residual(case)
