"""The small-batch kernel on exact codes (groups of 128; bfloat16 of 2 to 8 rows, fp16 of 17 to 64) against the oracle: last tiles
of rows and columns, fewer k blocks than wavefronts, remainders of the unrolled loop, one to sixteen row blocks per workgroup, and
calls that reach it by default."""
import numpy as np
import pytest

import synth_inputs
from test_gpu_bf16_e0m3 import assert_bf16_quantize_exact, bf_bits, bf_dev, check_bf16_matmul
from test_gpu_fused import check_fused
from test_gpu_parity import assert_quantize_exact, check_matmul, e0m4, to_dev, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture
def forced(e0m4):
    e0m4.e0m4_set_knob("gemv_mfma", 7)
    yield
    e0m4.e0m4_set_knob("gemv_mfma", 0)
    e0m4.e0m4_set_knob("gemv_workgroups", 0)


# N, K, workgroups aimed at: 1, 2, 3 and 4 row blocks per wavefront, one, two and four groups of wavefronts
@pytest.mark.parametrize("N,K,workgroups", [(17, 128, 0), (203, 1152, 0), (333, 2176, 12), (520, 1664, 4), (260, 640, 1), (1000, 4224, 9)])
@pytest.mark.parametrize("fmt,M", [("bf16", M) for M in (2, 4, 5, 8)] + [("e0m4", M) for M in (17, 32, 33, 48, 49, 64)])
def test_plain(e0m4, oracle, forced, fmt, M, N, K, workgroups):
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    if fmt == "bf16":
        codes, What, (oc, os_, ob) = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=7000 + N), 128)
        X = synth_inputs.activations_bf16(M, K, seed=7100 + M)
        X[0] = 0
        X[0, 77] = 0x3FC0                               # one row with a single 1.5: 1.5 scale (w1 - bias), rounded once
        Y = e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, 128)
        Yref, absdot = oracle.bf16_matmul(X, What)
        check_bf16_matmul(oracle, Y, Yref, absdot, "bf16 M=%d" % M)
        exact = 1.5 * oracle.bf16_to_float64(os_[:, 0]) * (2 + oc[:, 77] / 8.0 - oracle.bf16_to_float64(ob[:, 0]))
        assert np.array_equal(bf_bits(Y)[0] & 0x7FFF, synth_inputs.to_bf16_bits(exact.astype(np.float32)) & 0x7FFF)
        return
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=7000 + N), 128)
    X = synth_inputs.activations(M, K, seed=7100 + M, outlier_frac=0.01)
    Y, Y2 = (e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, 128) for _ in range(2))
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(Y, Yref, absdot, "M=%d" % M)
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("N,K", [(448, 1664), (1088, 4096), (27392, 256)])
@pytest.mark.parametrize("M", [3, 17, 24, 33, 48, 49, 64])
def test_default_choice(e0m4, oracle, M, N, K):
    # the fused entry point without operators gives the same bits (where the plain call does not multiply rounded weights, as with
    # 27392 x 256), and with a residual it has the workspace that it needs
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=7400), 128)
    X = synth_inputs.activations(M, K, seed=7500 + M)
    Y = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, 128)
    Y2 = e0m4.e0m4_matmul_fused(to_dev(X), codes, N, K, 128)
    assert N > 2000 or torch.equal(Y, Y2)
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(Y, Yref, absdot, "M=%d" % M)
    R = synth_inputs.activations(M, N, seed=7600 + M)
    YR = e0m4.e0m4_matmul_fused(to_dev(X), codes, N, K, 128, residual=to_dev(R))
    YRref, info = oracle.matmul_fused(X, What, residual=R)
    check_fused(YR, YRref, info, False, False, "residual M=%d" % M)


# calls whose chunks have a compute unit (or a place on one) each stay on them, to the bit, as in the last case four chunks in two
# rounds; the others take exact codes
@pytest.mark.parametrize("M,N,K,exact", [(59, 840, 4096, False), (17, 1550, 6144, False), (24, 904, 2688, False), (32, 576, 2304, True),
                                         (28, 1904, 3328, True), (28, 800, 3328, False),
                                         (35, 1816, 2688, False), (20, 2856, 2432, True), (47, 2376, 1920, True), (24, 4608, 1536, True),
                                         (51, 2040, 4096, False), (64, 2832, 3712, True)])
def test_chunks_where_they_are_faster(e0m4, oracle, M, N, K, exact):
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=7700), 128)
    X = synth_inputs.activations(M, K, seed=7800 + M, outlier_frac=0.01)
    Y = {}
    try:
        for mode in (0, 7, 8):
            e0m4.e0m4_set_knob("gemv_mfma", mode)
            Y[mode] = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, 128)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(Y[0], Yref, absdot, "M=%d" % M)
    assert not torch.equal(Y[7], Y[8])                  # (two orders of the sums)
    assert torch.equal(Y[0], Y[7 if exact else 8])


# bfloat16: with three and four row blocks per wavefront not where these lie almost a multiple of 16 KiB apart (to the bits of the
# staging kernel there)
@pytest.mark.parametrize("workgroups,N,K,exact", [(3, 190, 1920, False), (3, 190, 1792, True), (2, 96, 3840, False), (2, 96, 7680, True),
                                                  (3, 96, 1920, True), (1, 128, 5760, False)])
def test_bf16_row_blocks_on_the_same_channels(e0m4, oracle, workgroups, N, K, exact):
    W, X, half = synth_inputs.weights_bf16(N, K, seed=7900), synth_inputs.activations_bf16(5, K, seed=7950), K // 256 * 128
    W[:, half:2 * half], X[:, half:2 * half], X[:, 2 * half:] = W[:, :half], X[:, :half] ^ 0x8000, 0
    codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, W, 128)       # (sums that cancel: what is left shows their order)
    Y = {}
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        for mode in (0, 7, 8):
            e0m4.e0m4_set_knob("gemv_mfma", mode)
            Y[mode] = e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, 128)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)
    Yref, absdot = oracle.bf16_matmul(X, What)
    check_bf16_matmul(oracle, Y[0], Yref, absdot, "K=%d" % K)
    assert torch.equal(Y[0].view(torch.int16), Y[7 if exact else 8].view(torch.int16))
    assert not torch.equal(Y[7].view(torch.int16), Y[8].view(torch.int16))
