"""The small-batch kernel with dequantised weight operands (plain matmuls, 2 <= M <= 128) against the CPU oracle, in the three
formats it serves: last tiles of 16 rows of X and 16 weight rows, k blocks that K does not fill, fewer k blocks than
wavefronts and remainders of the unrolled loop, one to sixteen row blocks per workgroup."""
import numpy as np
import pytest

import synth_inputs
from test_gpu_bf16_e0m3 import assert_bf16_quantize_exact, bf_bits, bf_dev, check_bf16_matmul
from test_gpu_parity import assert_quantize_exact, check_matmul, e0m4, to_dev, torch  # noqa: F401
import test_gpu_e0m8

pytestmark = pytest.mark.gpu

# N, K, group, workgroups aimed at: 1, 2, 3 and 4 row blocks per wavefront, one, two and four groups of wavefronts
SHAPES = [(17, 128, 64, 0), (203, 1152, 64, 0), (333, 2176, 128, 12), (520, 1664, 128, 4), (260, 640, 64, 1), (1000, 4224, 128, 9)]


@pytest.mark.parametrize("fmt", ["e0m4", "e0m8", "bf16"])
@pytest.mark.parametrize("N,K,G,workgroups", SHAPES + [(203, 416, 32, 3), (48, 96, 32, 0)])
@pytest.mark.parametrize("M", [2, 9, 16, 17, 33, 48, 64, 65, 127])
def test_forced(e0m4, oracle, fmt, N, K, G, workgroups, M):
    if fmt == "e0m8" and G == 32:
        pytest.skip("8-bit codes have groups of 64 and 128")
    seed = 4000 + N + K
    e0m4.e0m4_set_knob("gemv_mfma", 4)
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        if fmt == "bf16":
            codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=seed), G)
            X = synth_inputs.activations_bf16(M, K, seed=seed + M)
            Y, Y2 = (e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G) for _ in range(2))
            Yref, absdot = oracle.bf16_matmul(X, What)
            check_bf16_matmul(oracle, Y, Yref, absdot, "bf16")
            assert np.array_equal(bf_bits(Y), bf_bits(Y2))
            return
        X = synth_inputs.activations(M, K, seed=seed + M, outlier_frac=0.01)
        W = synth_inputs.weights(N, K, seed=seed)
        if fmt == "e0m8":
            codes, What = test_gpu_e0m8.assert_quantize_exact(e0m4, oracle, W, G)
            Y, Y2 = (e0m4.e0m8_matmul(to_dev(X), codes, N, K, G) for _ in range(2))
        else:
            (codes, _, _), What = assert_quantize_exact(e0m4, oracle, W, G)
            Y, Y2 = (e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G) for _ in range(2))
        Yref, absdot = oracle.matmul(X, What)
        check_matmul(Y, Yref, absdot, fmt)
        assert torch.equal(Y, Y2)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)


@pytest.mark.parametrize("M", [3, 20])
def test_infinite_activation_stays_in_its_row(e0m4, oracle, M):
    # a k block that K does not fill: what stands in for the missing activations is zero, whatever the row holds
    N, K, G = 70, 160, 32
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=4900), G)
    X = synth_inputs.activations(M, K, seed=4901)
    X[1, 130] = np.inf
    e0m4.e0m4_set_knob("gemv_mfma", 4)
    try:
        Y = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G).cpu().numpy()
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
    X[1, 130] = 0
    keep = np.arange(M) != 1
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(torch.from_numpy(Y[keep]), Yref[keep], absdot[keep], "rows without the infinity")
    w = What[:, 130].astype(np.float64)
    assert np.array_equal(Y[1][w != 0], (np.sign(w[w != 0]) * np.inf).astype(np.float16)) and np.isnan(Y[1][w == 0]).all()


@pytest.mark.parametrize("N,K,G,workgroups", SHAPES + [(203, 416, 32, 3), (48, 96, 32, 0)])
@pytest.mark.parametrize("M", [3, 4, 5, 8])
def test_few_rows_of_a_tile(e0m4, oracle, M, N, K, G, workgroups):
    # up to four and up to eight rows only these are loaded: the bits of the same rows among sixteen, which add in one order
    (codes, _, _), What = assert_quantize_exact(e0m4, oracle, synth_inputs.weights(N, K, seed=4950 + N), G)
    X = synth_inputs.activations(16, K, seed=4960 + K, outlier_frac=0.01)
    e0m4.e0m4_set_knob("gemv_mfma", 4)
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        Y16 = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G)
        Y = e0m4.e0m4_matmul(to_dev(X[:M]), codes, None, None, N, K, G)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)
    Yref, absdot = oracle.matmul(X[:M], What)
    check_matmul(Y, Yref, absdot, "M=%d" % M)
    assert torch.equal(Y, Y16[:M])


# five row blocks per wavefront (three with exact codes and four tiles of X), one to seven k blocks per wavefront and a last one
# that K does not fill
@pytest.mark.parametrize("fmt,M", [("e0m4", 16), ("e0m4", 48), ("bf16", 17), ("bf16", 33), ("e0m8", 48), ("exact", 49), ("exact", 64)])
@pytest.mark.parametrize("K", [256, 1088, 2176, 3200, 6272])
def test_most_row_blocks_per_wavefront(e0m4, oracle, fmt, M, K):
    N, workgroups, G = (380, 5, 64) if fmt != "exact" else (333, 7, 128)
    if K % G:
        pytest.skip("K is not whole groups")
    e0m4.e0m4_set_knob("gemv_mfma", 7 if fmt == "exact" else 4)
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        if fmt == "bf16":
            codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=4970 + K), G)
            X = synth_inputs.activations_bf16(M, K, seed=4980 + M)
            Y = e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G)
            check_bf16_matmul(oracle, Y, *oracle.bf16_matmul(X, What), "bf16")
            return
        X, W = synth_inputs.activations(M, K, seed=4980 + M, outlier_frac=0.01), synth_inputs.weights(N, K, seed=4970 + K)
        if fmt == "e0m8":
            codes, What = test_gpu_e0m8.assert_quantize_exact(e0m4, oracle, W, G)
            Y = e0m4.e0m8_matmul(to_dev(X), codes, N, K, G)
        else:
            (codes, _, _), What = assert_quantize_exact(e0m4, oracle, W, G)
            Y = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G)
        check_matmul(Y, *oracle.matmul(X, What), fmt)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)


# (wide weights: on either side of the number of row blocks per compute unit up to which this kernel is faster than the GEMM)
@pytest.mark.parametrize("fmt,M,N,K,norm,here", [
    ("e0m4", 32, 24576, 512, True, True), ("e0m4", 32, 24592, 512, True, False), ("e0m4", 17, 49152, 768, True, True),
    ("e0m4", 32, 49168, 896, True, False), ("e0m4", 32, 49168, 1536, False, True), ("e0m4", 20, 98304, 1024, True, True), ("e0m4", 24, 98320, 1536, False, False),
    ("e0m4", 48, 24576, 512, True, True), ("e0m4", 33, 24592, 512, True, False), ("e0m4", 48, 40960, 512, True, True),
    ("e0m4", 40, 40976, 2048, False, False), ("e0m4", 64, 16384, 768, True, True), ("e0m4", 64, 16400, 768, True, False),
    ("e0m8", 32, 53248, 256, True, True), ("e0m8", 32, 53264, 384, True, False), ("e0m8", 32, 53264, 512, True, True), ("e0m8", 17, 81936, 512, True, False), ("e0m8", 40, 16400, 896, True, False),
    ("e0m8", 40, 40960, 1024, True, True), ("e0m8", 40, 40976, 2560, False, False), ("e0m8", 64, 16384, 256, True, True),
    ("e0m8", 64, 16400, 256, True, False)])
def test_wide_weights_go_where_they_are_faster(e0m4, fmt, M, N, K, norm, here):
    G = 64 if fmt == "e0m4" else 128
    quantize = e0m4.e0m4_quantize if fmt == "e0m4" else e0m4.e0m8_quantize
    codes = quantize(to_dev(synth_inputs.weights(512, K, seed=5000)).repeat(-(-N // 512), 1)[:N].contiguous(), G)[0]
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=5001, outlier_frac=0.01)), to_dev(synth_inputs.norm_weight(K, 5002))

    def run(mode):
        e0m4.e0m4_set_knob("gemv_mfma", mode)
        try:
            if norm:
                return (e0m4.e0m4_matmul_fused if fmt == "e0m4" else e0m4.e0m8_matmul_fused)(X, codes, N, K, G, rms_gamma=gamma, rms_eps=1e-5)
            return e0m4.e0m4_matmul(X, codes, None, None, N, K, G) if fmt == "e0m4" else e0m4.e0m8_matmul(X, codes, N, K, G)
        finally:
            e0m4.e0m4_set_knob("gemv_mfma", 0)

    by_default, small_batch, gemm = run(0), run(4), run(5)
    assert not torch.equal(small_batch, gemm)           # (they add in different orders)
    assert torch.equal(by_default, small_batch if here else gemm)


# rows of one to eight k blocks: one, two and four groups of wavefronts, the last with fewer row blocks than the others or none
@pytest.mark.parametrize("fmt,K", [("e0m4", 96), ("e0m4", 256), ("e0m4", 512), ("e0m4", 640), ("bf16", 128), ("bf16", 384), ("bf16", 512),
                                   ("e0m8", 64), ("e0m8", 128), ("e0m8", 256), ("e0m8", 320), ("exact", 128), ("exact", 256), ("exact", 512)])
@pytest.mark.parametrize("M", [5, 17, 49, 64])
def test_short_rows(e0m4, oracle, fmt, K, M):
    G = 32 if K % 64 else 64 if fmt != "exact" else 128
    if fmt == "exact" and M <= 16:
        pytest.skip("17 rows and more")
    for N, workgroups in ((16 * 9 - 3, 9), (333, 7), (16 * 25, 5), (16 * 13, 1)):
        e0m4.e0m4_set_knob("gemv_mfma", 7 if fmt == "exact" else 4)
        e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
        try:
            if fmt == "bf16":
                codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=5010 + K), G)
                X = synth_inputs.activations_bf16(M, K, seed=5020 + M)
                check_bf16_matmul(oracle, e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G), *oracle.bf16_matmul(X, What), "bf16")
                continue
            X, W = synth_inputs.activations(M, K, seed=5020 + M, outlier_frac=0.01), synth_inputs.weights(N, K, seed=5010 + K)
            if fmt == "e0m8":
                codes, What = test_gpu_e0m8.assert_quantize_exact(e0m4, oracle, W, G)
                Y = e0m4.e0m8_matmul(to_dev(X), codes, N, K, G)
            else:
                (codes, _, _), What = assert_quantize_exact(e0m4, oracle, W, G)
                Y = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G)
            check_matmul(Y, *oracle.matmul(X, What), fmt)
        finally:
            e0m4.e0m4_set_knob("gemv_mfma", 0)
            e0m4.e0m4_set_knob("gemv_workgroups", 0)
