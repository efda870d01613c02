"""GEMM tiles of 128 columns, whose wavefronts hold one block of 32 columns: last tiles of rows and columns, row lengths that are no
multiple of 8, the gated product of two wavefronts' sums in whole tiles and in K splits, a K range shorter than the pipeline, every
group and format; K quarters inside a workgroup; the same bits as the tiles of 256 columns in the same number of splits; and the number of K splits, hence the
bits, of fused calls of up to 64 rows by default routes."""
import ctypes

import pytest

import synth_inputs
from test_gpu_bf16_e0m3 import assert_bf16_quantize_exact, bf_dev, check_bf16_matmul
from test_gpu_fused import COMBOS, e0m4, quantized, run_fused, to_dev, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def with_knobs(e0m4, fn, **knobs):
    for k, v in knobs.items():
        e0m4.e0m4_set_knob(k, v)
    try:
        return fn()
    finally:
        for k in knobs:
            e0m4.e0m4_set_knob(k, 0)


@pytest.mark.parametrize("variant", [3, 6])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("norm,swiglu,res", COMBOS)
def test_against_the_oracle(e0m4, oracle, variant, splits, norm, swiglu, res):
    for M, N, K, G, bits in ((300, 640, 1024, 128, 4), (9, 192, 384, 64, 4), (130, 1088, 512, 32, 4), (65, 128, 128, 128, 4), (129, 704, 640, 128, 8)):
        with_knobs(e0m4, lambda: run_fused(e0m4, oracle, M, N, K, G, seed=1400 + M, norm=norm, swiglu=swiglu, res=res, outliers=True, bits=bits),
                   gemm_variant=variant, gemm_splits=splits, gemv_mfma=1)


@pytest.mark.parametrize("M,N,K", [(64, 192, 1024), (200, 327, 640), (257, 576, 2048), (129, 1152, 128)])
def test_bits_of_the_wide_tiles(e0m4, oracle, M, N, K):
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=1420 + N)
    X = to_dev(synth_inputs.activations(M, K, seed=1421 + M, outlier_frac=0.01))
    for swiglu in (False, True):
        if swiglu and N % 64:
            continue
        R = to_dev(synth_inputs.residual(M, N // 2 if swiglu else N, 1422))
        for splits in (1, 2):
            Y = [with_knobs(e0m4, lambda: e0m4.e0m4_matmul_fused(X, codes, N, K, 128, residual=R, epilogue=1 if swiglu else 0),
                            gemm_variant=v, gemm_splits=splits, gemv_mfma=1) for v in (4, 6, 3)]
            assert torch.equal(Y[0], Y[1]) and torch.equal(Y[0], Y[2]), (swiglu, splits)


# (K splits as by 64 x 256 tiles: the most, fewer, and as many tiles as compute units)
@pytest.mark.parametrize("N,K,splits", [(1536, 5888, 8), (4096, 13696, 8), (9216, 3072, 6), (27392, 4096, 4), (65536, 1024, 1)])
def test_fused_calls_of_few_rows_keep_their_splits(e0m4, N, K, splits):
    M = 45
    codes = e0m4.e0m4_quantize(to_dev(synth_inputs.weights(256, K, seed=1431)).repeat(N // 256, 1), 128)[0]
    X, R = to_dev(synth_inputs.activations(M, K, seed=1432)), to_dev(synth_inputs.residual(M, N, 1433))
    forced = with_knobs(e0m4, lambda: e0m4.e0m4_matmul_fused(X, codes, N, K, 128, residual=R), gemm_variant=4, gemm_splits=splits, gemv_mfma=1)
    by_default = with_knobs(e0m4, lambda: e0m4.e0m4_matmul_fused(X, codes, N, K, 128, residual=R), gemv_mfma=1)
    assert torch.equal(forced, by_default)


@pytest.mark.parametrize("variant", [3, 6])
@pytest.mark.parametrize("M,N,K,G", [(300, 600, 1024, 128), (129, 272, 384, 32), (65, 203, 2048, 64), (64, 128, 128, 64)])
def test_bf16(e0m4, oracle, variant, M, N, K, G):
    codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=1440 + N + K), G)
    X = synth_inputs.activations_bf16(M, K, seed=1441 + M)
    Y = with_knobs(e0m4, lambda: e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G), gemm_variant=variant)
    Yref, absdot = oracle.bf16_matmul(X, What)
    check_bf16_matmul(oracle, Y, Yref, absdot, "bf16 gemm variant %d M=%d N=%d K=%d" % (variant, M, N, K))


# (calls with four K splits; quarters of equal and unequal length, ragged last tiles, every group)
@pytest.mark.parametrize("N,K,G", [(11392, 2048, 128), (12352, 2176, 128), (14400, 2048, 32), (12224, 2304, 64)])
@pytest.mark.parametrize("M", [33, 64])
def test_bits_of_k_quarters(e0m4, M, N, K, G):
    codes = e0m4.e0m4_quantize(to_dev(synth_inputs.weights(64, K, seed=1450)).repeat((N + 63) // 64, 1)[:N].contiguous(), G)[0]
    X = to_dev(synth_inputs.activations(M, K, seed=1451 + M, outlier_frac=0.01))
    assert with_knobs(e0m4, lambda: e0m4.e0m4_fused_workspace_bytes(M, N, K, G, False, 0), gemv_mfma=1) == 4 * M * N * 4
    for swiglu, res in ((True, False), (False, True), (True, True)):
        if swiglu and N % 64:
            continue
        R = to_dev(synth_inputs.residual(M, N // 2 if swiglu else N, 1452)) if res else None
        Y = [with_knobs(e0m4, lambda: e0m4.e0m4_matmul_fused(X, codes, N, K, G, residual=R, epilogue=1 if swiglu else 0), gemv_mfma=1, **k)
             for k in ({"gemm_variant": 4, "gemm_splits": 4}, {"gemm_variant": 7})]
        assert torch.equal(*Y), (swiglu, res)


# (8-bit codes, up to 64 rows, at most a work item per compute unit: splits of one pair of K slices and more, equal and unequal)
@pytest.mark.parametrize("N,K,splits", [(832, 512, 4), (600, 1152, 2), (320, 2176, 8), (64, 384, 3)])
@pytest.mark.parametrize("swiglu,res", [(True, False), (False, True), (True, True)])
def test_8bit_codes_two_slices_ahead(e0m4, oracle, N, K, splits, swiglu, res):
    if swiglu and N % 64:
        N -= N % 64
    for M in (19, 64):
        with_knobs(e0m4, lambda: run_fused(e0m4, oracle, M, N, K, 128, seed=1460 + M, norm=False, swiglu=swiglu, res=res, outliers=True, bits=8),
                   gemm_variant=4, gemm_splits=splits, gemv_mfma=1)


# (large weights whose work items would be more than the compute units in splits: whole 64 x 128 tiles, whose sums are in another order)
@pytest.mark.parametrize("bits,M,N,K,splits", [(8, 63, 27456, 2816, 4), (4, 56, 26112, 2560, 5)])
def test_calls_with_an_rms_norm_alone_choose_their_splits(e0m4, bits, M, N, K, splits):
    quantize, fused = (e0m4.e0m8_quantize, e0m4.e0m8_matmul_fused) if bits == 8 else (e0m4.e0m4_quantize, e0m4.e0m4_matmul_fused)
    codes = quantize(to_dev(synth_inputs.weights(192, K, seed=1470)).repeat(N // 192, 1), 128)[0]
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=1471, outlier_frac=0.01)), to_dev(synth_inputs.norm_weight(K, 1472))

    def run(**knobs):
        return with_knobs(e0m4, lambda: fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5), **knobs)

    by_default, whole, split = run(), run(gemm_variant=6, gemm_splits=1), run(gemm_variant=4, gemm_splits=splits)
    assert torch.equal(by_default, whole) and not torch.equal(by_default, split)


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3), ("params", ctypes.c_void_p),
                ("shared", ctypes.c_uint)]


def launches(fn):
    """Workgroups, threads and LDS of the kernels that a call launches, which tell the GEMM's tiles apart."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    fn()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fn()
    hip, n = ctypes.CDLL("libamdhip64.so"), ctypes.c_size_t(0)
    raw = ctypes.c_void_p(graph.raw_cuda_graph())
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = KernelNodeParams()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append((p.grid.x, p.block.x, p.shared))
    return out


# (the tile of a gated call by default: on tiles of 128 columns its epilogue takes longer; tiles of 128 x 256 that are more than the compute
# units, the last row of them short)
@pytest.mark.parametrize("bits,M,N,K,tiles", [(4, 609, 10816, 384, (4, 5)), (4, 222, 8640, 256, (4,)), (8, 732, 9600, 256, (4, 5)), (8, 121, 21056, 384, (4,)),
                                              (4, 107, 10368, 768, (6,)), (4, 439, 17920, 2432, (4,)), (8, 391, 17344, 2944, (4,)), (4, 288, 23296, 640, (4,)),
                                              (8, 142, 200192, 1920, (4,)), (4, 39, 36096, 128, (4,)), (4, 60, 33216, 256, (4,)), (8, 46, 37056, 128, (4,)), (8, 20, 44480, 256, (4,)), (4, 34, 32768, 384, (6,))])
def test_tiles_of_gated_calls(e0m4, bits, M, N, K, tiles):
    quantize, fused = (e0m4.e0m8_quantize, e0m4.e0m8_matmul_fused) if bits == 8 else (e0m4.e0m4_quantize, e0m4.e0m4_matmul_fused)
    codes = quantize(to_dev(synth_inputs.weights(64, K, seed=1480)).repeat(-(-N // 64), 1)[:N].contiguous(), 128)[0]
    X = to_dev(synth_inputs.activations(M, K, seed=1481))
    Y = X.new_empty((M, N // 2))

    def run(**knobs):
        return with_knobs(e0m4, lambda: launches(lambda: fused(X, codes, N, K, 128, epilogue=1, out=Y)), **knobs)

    by_default = run()
    assert by_default in [run(gemm_variant=v, gemm_splits=1) for v in tiles], by_default


def test_a_tie_between_whole_tiles_and_splits_is_the_whole_tiles(e0m4):
    M, N, K = 2048, 5120, 13696
    codes = e0m4.e0m4_quantize(to_dev(synth_inputs.weights(64, K, seed=1490)).repeat(N // 64, 1), 64)[0]
    X, R = to_dev(synth_inputs.activations(M, K, seed=1491)), to_dev(synth_inputs.residual(M, N, 1492))
    Y = torch.empty_like(R)

    def run(**knobs):
        return with_knobs(e0m4, lambda: launches(lambda: e0m4.e0m4_matmul_fused(X, codes, N, K, 64, residual=R, out=Y)), **knobs)

    assert run() == run(gemm_variant=2, gemm_splits=1)
