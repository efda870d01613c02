"""Few rows of X on long rows of weights (2 <= M <= 16, X larger than the LDS, one row block per workgroup): the kernel that takes
X block by block gives the bits of the one that stages it in phases, and both are the oracle's within its bar."""
import numpy as np
import pytest

import synth_inputs
from test_gpu_parity import assert_quantize_exact, check_matmul, e0m4, to_dev, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [4, 5, 8, 9, 16])
@pytest.mark.parametrize("N,K", [(130, 16384), (17, 9728), (203, 13696), (64, 24704), (48, 49152)])
def test_same_bits_as_in_phases(e0m4, oracle, M, N, K):
    # (24704: 49 work items, the last of one block; 49152: the most items that the kernel takes)
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=5000 + N), 128)
    X = synth_inputs.activations(M, K, seed=5100 + M, outlier_frac=0.01)
    R = synth_inputs.activations(M, N, seed=5200 + M)
    Y, YR = [], []
    try:
        for mode in (0, 2):
            e0m4.e0m4_set_knob("gemv_mfma", mode)
            Y.append(e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, 128))
            YR.append(e0m4.e0m4_matmul_fused(to_dev(X), codes, N, K, 128, residual=to_dev(R)))
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(Y[0], Yref, absdot, "M=%d K=%d" % (M, K))
    assert torch.equal(Y[0].view(torch.int16), Y[1].view(torch.int16))
    assert torch.equal(YR[0].view(torch.int16), YR[1].view(torch.int16))
