"""Fused matmuls of up to 64 rows by default routes against the oracle: an rms-norm alone runs before the kernel with dequantised
operands, other operators on chunks of rows or the GEMM."""
import pytest

from test_gpu_fused import COMBOS, e0m4, run_fused  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm,swiglu,res", COMBOS)
@pytest.mark.parametrize("M,N,K,G,bits", [(9, 1088, 1664, 64, 4), (16, 448, 672, 32, 4), (30, 5120, 1536, 64, 4), (45, 4608, 2048, 128, 4),
                                          (48, 832, 160, 32, 4), (64, 4608, 1152, 128, 4), (30, 4608, 2304, 128, 8), (64, 2048, 1152, 64, 8)])
def test_by_default(e0m4, oracle, M, N, K, G, bits, norm, swiglu, res):
    run_fused(e0m4, oracle, M, N, K, G, seed=950 + M, norm=norm, swiglu=swiglu, res=res, outliers=True, bits=bits)
