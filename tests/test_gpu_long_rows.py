"""Few rows of X with one or two row blocks per workgroup: the kernel that takes X block by block gives the bits of the one that
stages it, whole or in phases, and both are the oracle's within its bar."""
import pytest

import synth_inputs
import test_gpu_e0m8
from test_gpu_fused import check_fused, run_fused
from test_gpu_parity import assert_quantize_exact, check_matmul, e0m4, to_dev, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [4, 5, 8, 9, 16])
@pytest.mark.parametrize("N,K", [(130, 16384), (17, 9728), (203, 13696), (64, 24704), (48, 49152)])
def test_same_bits_as_in_phases(e0m4, oracle, M, N, K):
    # (24704: 49 work items, the last of one block; 49152: the most items that the kernel takes)
    same_bits(e0m4, oracle, M, N, K, 128, 0)


# three workgroups asked for: two row blocks in some of them, one in others; items that leave a remainder over eight and sixteen
# wavefronts, phases with and without one, a last phase of fewer items
@pytest.mark.parametrize("N,target", [(80, 3), (96, 3), (17, 0)])
@pytest.mark.parametrize("K", [1536, 2560, 5120, 5248, 8192, 13696, 16512])
@pytest.mark.parametrize("M,G", [(3, 128), (5, 128), (16, 128), (3, 64), (4, 64), (6, 64), (8, 64), (3, 32), (4, 32)])
def test_same_bits_as_staged(e0m4, oracle, M, G, K, N, target):
    same_bits(e0m4, oracle, M, N, K, G, target)


def same_bits(e0m4, oracle, M, N, K, G, target):
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=5000 + N), G)
    X = synth_inputs.activations(M, K, seed=5100 + M, outlier_frac=0.01)
    R = synth_inputs.activations(M, N, seed=5200 + M)

    def plain(x):
        return e0m4.e0m4_matmul(x, codes, None, None, N, K, G)

    def fused(x, **residual):
        return e0m4.e0m4_matmul_fused(x, codes, N, K, G, **residual)

    compare(e0m4, oracle, plain, fused, X, What, R, target)


def compare(e0m4, oracle, plain, fused, X, What, R, target):
    e0m4.e0m4_set_knob("gemv_workgroups", target)
    try:
        e0m4.e0m4_set_knob("gemv_mfma", 9)              # block by block wherever that can run, also where it does not pay
        Y, YR = plain(to_dev(X)), fused(to_dev(X), residual=to_dev(R))
        e0m4.e0m4_set_knob("gemv_mfma", 2)              # staged (plain calls in groups of 64 and 32 only through the fused entry point)
        Y2, YR2 = fused(to_dev(X)), fused(to_dev(X), residual=to_dev(R))
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)
    Yref, info = oracle.matmul_fused(X, What)
    check_matmul(Y, Yref, info["absdot"], "plain")
    YRref, info = oracle.matmul_fused(X, What, residual=R)
    check_fused(YR, YRref, info, False, False, "residual")
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))
    assert torch.equal(YR.view(torch.int16), YR2.view(torch.int16))


# The residual may be the output's own buffer (two row blocks in some workgroups with three asked for, one with none).
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("N,target,K", [(80, 3, 2560), (17, 0, 2560), (203, 0, 13696)])
@pytest.mark.parametrize("M", [5, 16])
def test_residual_in_place(e0m4, oracle, M, N, target, K, bits):
    e0m4.e0m4_set_knob("gemv_workgroups", target)
    e0m4.e0m4_set_knob("gemv_mfma", 9)
    try:
        Y, Y2 = (run_fused(e0m4, oracle, M, N, K, 128, seed=5600 + M, res=True, in_place=i, bits=bits) for i in (False, True))
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))


# 8-bit codes: k blocks of 64 weights, the same order of sums
@pytest.mark.parametrize("N,target", [(80, 3), (17, 0)])
@pytest.mark.parametrize("K", [768, 1344, 2560, 4096, 5184, 8192, 13696])
@pytest.mark.parametrize("M", [3, 5, 8, 9, 16])
def test_same_bits_as_staged_8bit(e0m4, oracle, M, K, N, target):
    codes, What = test_gpu_e0m8.assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=5300 + N), 64)
    X = synth_inputs.activations(M, K, seed=5400 + M, outlier_frac=0.01)
    R = synth_inputs.activations(M, N, seed=5500 + M)

    def plain(x):
        return e0m4.e0m8_matmul(x, codes, N, K, 64)

    def fused(x, **residual):
        return e0m4.e0m8_matmul_fused(x, codes, N, K, 64, **residual)

    compare(e0m4, oracle, plain, fused, X, What, R, target)
