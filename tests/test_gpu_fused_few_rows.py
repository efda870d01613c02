"""Fused matmuls of up to 64 rows: all rows in a workgroup, to the bits of the small-batch kernel on chunks of rows, with every
operator, over last tiles of rows and columns, one to four row blocks per workgroup, work items that wavefronts of the order have in
other row blocks and that end before their fourth k block; the calls that have no workspace for the normalised activations; and
calls by default routes against the oracle."""
import ctypes

import numpy as np
import pytest

import synth_inputs
from test_gpu_fused import COMBOS, e0m4, quantized, run_fused, to_dev, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def call(e0m4, mode, X, codes, N, K, gamma, swiglu, residual):
    e0m4.e0m4_set_knob("gemv_mfma", mode)
    try:
        return e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5, residual=residual,
                                      epilogue=e0m4.E0M4_EPILOGUE_SWIGLU if swiglu else e0m4.E0M4_EPILOGUE_NONE)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)


# N, K, workgroups aimed at: 1 to 4 and 7 row blocks per workgroup (gated: 2, 4 and 8); 1, 3, 4, 8, 9 and 14 work items
@pytest.mark.parametrize("N,K,workgroups", [(192, 128, 0), (448, 1664, 0), (320, 1152, 10), (1088, 2048, 34), (576, 4096, 12), (448, 1536, 7),
                                            (320, 4480, 20), (192, 7040, 6), (1728, 2304, 16)])
@pytest.mark.parametrize("M", [17, 32, 41, 48, 49, 64])
def test_bits_of_the_chunks(e0m4, oracle, M, N, K, workgroups):
    codes, What = quantized(e0m4, oracle, N, K, 128, seed=900 + N)
    gamma_h = synth_inputs.norm_weight(K, 902)
    X_h = synth_inputs.activations(M, K, seed=901 + M, outlier_frac=0.01)
    X, gamma = to_dev(X_h), to_dev(gamma_h)
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        for norm, swiglu, res in COMBOS + [(False, True, True), (True, True, False)]:
            R_h = synth_inputs.residual(M, N // 2 if swiglu else N, 903)
            Y, Yc = (call(e0m4, mode, X, codes, N, K, gamma if norm else None, swiglu, to_dev(R_h) if res else None) for mode in (7, 8))
            assert torch.equal(Y, Yc), (norm, swiglu, res)
            if res:                                     # the residual updated in place
                Z = to_dev(R_h)
                e0m4.e0m4_set_knob("gemv_mfma", 7)
                e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma if norm else None, rms_eps=1e-5, residual=Z, out=Z,
                                       epilogue=e0m4.E0M4_EPILOGUE_SWIGLU if swiglu else e0m4.E0M4_EPILOGUE_NONE)
                e0m4.e0m4_set_knob("gemv_mfma", 0)
                assert torch.equal(Z, Yc), (norm, swiglu)
        # (a matrix that ends in the middle of a row block)
        codes, _ = quantized(e0m4, oracle, N - 21, K, 128, seed=904 + N)
        R = to_dev(synth_inputs.residual(M, N - 21, 905))
        assert torch.equal(*(call(e0m4, mode, X, codes, N - 21, K, None, False, R) for mode in (7, 8)))
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)


@pytest.mark.parametrize("norm,swiglu,res", COMBOS)
@pytest.mark.parametrize("M,N,K,G,bits", [(9, 1088, 1664, 64, 4), (16, 448, 672, 32, 4), (30, 5120, 1536, 64, 4), (45, 4608, 2048, 128, 4),
                                          (48, 832, 160, 32, 4), (64, 4608, 1152, 128, 4), (30, 4608, 2304, 128, 8), (64, 2048, 1152, 64, 8)])
def test_by_default(e0m4, oracle, M, N, K, G, bits, norm, swiglu, res):
    run_fused(e0m4, oracle, M, N, K, G, seed=950 + M, norm=norm, swiglu=swiglu, res=res, outliers=True, bits=bits)


def test_without_a_workspace(e0m4, oracle):
    M, N, K = 45, 4608, 2048
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=970)
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=971)), to_dev(synth_inputs.norm_weight(K, 972))
    need = e0m4.lib().e0m4_fused_workspace_best_bytes(M, N, K, 128, 1, 0)
    assert need >= M * K * 2 and e0m4.e0m4_fused_workspace_bytes(M, N, K, 128, True, 0) == 0
    room = torch.full((need + 16,), 255, dtype=torch.uint8, device=X.device)
    for ws, nbytes in ((0, 0), (0, need), (room.data_ptr(), need - 1), (room.data_ptr() + 8, need)):
        Y = torch.empty((M, N), dtype=torch.float16, device=X.device)
        rc = e0m4.lib().e0m4_matmul_fused(X.data_ptr(), M, gamma.data_ptr(), ctypes.c_float(1e-5), codes.data_ptr(), N, K, 128, 0, 0,
                                          Y.data_ptr(), ws, nbytes, torch.cuda.current_stream().cuda_stream)
        assert rc == 0 and torch.equal(Y, call(e0m4, 8, X, codes, N, K, gamma, False, None))
    assert np.all(room.cpu().numpy() == 255)            # (nothing was written there)


def test_on_a_raw_stream_that_is_not_the_current_one(e0m4, oracle):
    """A workspace cannot be allocated for such a stream: calls that need none are served without, others say what is missing."""
    M, N, K = 45, 4608, 2048
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=980)
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=981)), to_dev(synth_inputs.norm_weight(K, 982))
    side = torch.cuda.Stream()
    Y = torch.empty((M, N), dtype=torch.float16, device=X.device)
    side.wait_stream(torch.cuda.current_stream())
    e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5, out=Y, stream=side.cuda_stream)
    side.synchronize()
    assert torch.equal(Y, e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5))
    X = to_dev(synth_inputs.activations(200, K, seed=983))
    with pytest.raises(ValueError, match="workspace"):
        e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5, out=X.new_empty((200, N)), stream=side.cuda_stream)


def test_a_workspace_that_is_not_needed_is_not_touched(e0m4, oracle):
    """A buffer that several calls share stays as it is where the call's stated need is 0."""
    M, N, K = 45, 4608, 2048
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=990)
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=991)), to_dev(synth_inputs.norm_weight(K, 992))
    room = torch.full((M * K * 2 + 256,), 255, dtype=torch.uint8, device=X.device)
    L, stream = e0m4.lib(), torch.cuda.current_stream().cuda_stream
    Y = torch.empty((2, M, N), dtype=torch.float16, device=X.device)

    def args(y):
        return (X.data_ptr(), M, gamma.data_ptr(), ctypes.c_float(1e-5), codes.data_ptr(), N, K, 128, 0, 0, y.data_ptr(),
                room.data_ptr(), room.numel(), stream)

    assert e0m4.e0m4_fused_workspace_bytes(M, N, K, 128, True, 0) == 0
    assert L.e0m4_matmul_fused(*args(Y[0])) == 0
    e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5, workspace=room)
    assert np.all(room.cpu().numpy() == 255)
    assert L.e0m4_matmul_fused_best(*args(Y[1])) == 0 and torch.equal(Y[0], Y[1])
    assert np.any(room.cpu().numpy() != 255)            # (the normalised activations)


@pytest.mark.parametrize("M,N,K,swiglu,brings", [(24, 2048, 2048, True, False), (26, 4096, 4608, True, False), (26, 4096, 4736, True, True),
                                                 (32, 4096, 1024, True, False), (32, 4160, 1024, True, True), (45, 4608, 2048, False, True)])
def test_calls_issued_one_by_one_allocate_only_where_that_is_the_faster_way(e0m4, oracle, M, N, K, swiglu, brings):
    codes = e0m4.e0m4_quantize(to_dev(synth_inputs.weights(64, K, seed=1000)).repeat(N // 64, 1), 128)[0]
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=1001, outlier_frac=0.01)), to_dev(synth_inputs.norm_weight(K, 1002))
    n_out = N // 2 if swiglu else N
    Y, Z = (torch.empty((M, n_out), dtype=torch.float16, device=X.device) for _ in range(2))

    def run(out, stream=None):
        e0m4.e0m4_matmul_fused(X, codes, N, K, 128, rms_gamma=gamma, rms_eps=1e-5, epilogue=1 if swiglu else 0, out=out, stream=stream)

    def allocations():
        return torch.cuda.memory_stats(X.device)["allocation.all.allocated"]

    before = allocations()
    run(Y)
    assert allocations() - before == (1 if brings else 0)
    graph = torch.cuda.CUDAGraph()                      # in a graph always, to the same bits
    with torch.cuda.graph(graph):
        before = allocations()
        run(Z)
        run(Z, torch.cuda.current_stream())
        assert allocations() - before == 2
    for _ in range(3):
        Z.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, Z)


# the shapes of test_bits_of_the_chunks with an rms-norm, whose calls from Python go in chunks where these are few
@pytest.mark.parametrize("N,K,workgroups", [(192, 128, 0), (448, 1664, 0), (320, 1152, 10), (1088, 2048, 34), (576, 4096, 12), (448, 1536, 7),
                                            (320, 4480, 20), (192, 7040, 6), (1728, 2304, 16)])
@pytest.mark.parametrize("M", [17, 32, 41, 48, 49, 64])
def test_bits_of_the_chunks_with_an_rms_norm(e0m4, oracle, M, N, K, workgroups):
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=900 + N)
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=901 + M, outlier_frac=0.01)), to_dev(synth_inputs.norm_weight(K, 902))
    e0m4.e0m4_set_knob("gemv_workgroups", workgroups)
    try:
        room = torch.empty(M * K * 2 + 256 + e0m4.e0m4_fused_workspace_bytes(M, N, K, 128, True, 0), dtype=torch.uint8, device=X.device)
        for swiglu, res in ((False, False), (False, True), (True, False), (True, True)):
            n_out = N // 2 if swiglu else N
            R = to_dev(synth_inputs.residual(M, n_out, 903)) if res else None
            Yc = call(e0m4, 8, X, codes, N, K, gamma, swiglu, R)
            Y = R.clone() if res else torch.empty_like(Yc)                     # (the residual updated in place)
            e0m4.e0m4_set_knob("gemv_mfma", 7)
            rc = e0m4.lib().e0m4_matmul_fused_best(X.data_ptr(), M, gamma.data_ptr(), ctypes.c_float(1e-5), codes.data_ptr(), N, K, 128,
                                                   1 if swiglu else 0, Y.data_ptr() if res else 0, Y.data_ptr(), room.data_ptr(), room.numel(),
                                                   torch.cuda.current_stream().cuda_stream)
            assert rc == 0 and torch.equal(Y, Yc), (swiglu, res)
    finally:
        e0m4.e0m4_set_knob("gemv_mfma", 0)
        e0m4.e0m4_set_knob("gemv_workgroups", 0)


# (two, three and four chunks, on either side of as many chunks as compute units)
@pytest.mark.parametrize("M,N,swiglu", [(20, 2048, False), (30, 2048, False), (45, 1024, False), (48, 1360, False), (48, 1376, False), (51, 1024, False),
                                        (64, 1024, False), (64, 1040, False), (24, 2048, True), (45, 1024, True), (45, 4096, True)])
def test_the_best_workspace_is_asked_for_where_it_is_used(e0m4, oracle, M, N, swiglu):
    K, epilogue = 1152, 1 if swiglu else 0
    codes, _ = quantized(e0m4, oracle, N, K, 128, seed=1010)
    X, gamma = to_dev(synth_inputs.activations(M, K, seed=1011)), to_dev(synth_inputs.norm_weight(K, 1012))
    room = torch.full((M * K * 2 + 256,), 255, dtype=torch.uint8, device=X.device)
    best = e0m4.lib().e0m4_fused_workspace_best_bytes(M, N, K, 128, 1, epilogue)
    assert best in (0, (M * K * 2 + 255) // 256 * 256) and e0m4.e0m4_fused_workspace_bytes(M, N, K, 128, True, epilogue) == 0
    Y = torch.empty((M, N // 2 if swiglu else N), dtype=torch.float16, device=X.device)
    rc = e0m4.lib().e0m4_matmul_fused_best(X.data_ptr(), M, gamma.data_ptr(), ctypes.c_float(1e-5), codes.data_ptr(), N, K, 128, epilogue, 0,
                                           Y.data_ptr(), room.data_ptr(), room.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and bool((room != 255).any()) == (best > 0)
    assert torch.equal(Y, call(e0m4, 8, X, codes, N, K, gamma, swiglu, None))
