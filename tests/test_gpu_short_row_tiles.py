"""Prompts whose last row tile of 128 holds 64 rows or fewer: those tiles are computed in two blocks of 32 rows and numbered behind
the whole ones (32776 and, gated, 32768 columns: as many tiles as compute units; 200: too few for that)."""
import numpy as np
import pytest

import synth_inputs
from test_gpu_bf16_e0m3 import assert_bf16_quantize_exact, bf_dev, check_bf16_matmul
from test_gpu_fused import run_fused
from test_gpu_parity import assert_quantize_exact, check_matmul, e0m4, to_dev, torch  # noqa: F401
import test_gpu_e0m8

pytestmark = pytest.mark.gpu

MS = [129, 192, 300]


@pytest.fixture(autouse=True)
def half_tiles(e0m4):
    e0m4.e0m4_set_knob("gemm_variant", 5)
    e0m4.e0m4_set_knob("gemm_splits", 1)
    yield
    e0m4.e0m4_set_knob("gemm_variant", 0)
    e0m4.e0m4_set_knob("gemm_splits", 0)


@pytest.mark.parametrize("fmt,G", [("e0m4", 32), ("e0m4", 64), ("e0m4", 128), ("e0m8", 128), ("bf16", 64)])
@pytest.mark.parametrize("N,K", [(200, 384), (32776, 128)])
@pytest.mark.parametrize("M", MS)
def test_plain(e0m4, oracle, M, N, K, fmt, G):
    if fmt == "bf16":
        codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=6000 + N), G)
        X = synth_inputs.activations_bf16(M, K, seed=6100 + M)
        Yref, absdot = oracle.bf16_matmul(X, What)
        check_bf16_matmul(oracle, e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G), Yref, absdot, "bf16 M=%d" % M)
        return
    W = synth_inputs.weights(N, K, seed=6000 + N)
    X = synth_inputs.activations(M, K, seed=6100 + M, outlier_frac=0.01)
    if fmt == "e0m8":
        codes, What = test_gpu_e0m8.assert_quantize_exact(e0m4, oracle, W, G)
        Y = e0m4.e0m8_matmul(to_dev(X), codes, N, K, G)
    else:
        (codes, _, _), What = assert_quantize_exact(e0m4, oracle, W, G)
        Y = e0m4.e0m4_matmul(to_dev(X), codes, None, None, N, K, G)
    Yref, absdot = oracle.matmul(X, What)
    check_matmul(Y, Yref, absdot, "%s M=%d" % (fmt, M))
    ones = np.ones_like(X)                              # (a row left out or taken twice would show in equal rows)
    Y1 = e0m4.e0m8_matmul(to_dev(ones), codes, N, K, G) if fmt == "e0m8" else e0m4.e0m4_matmul(to_dev(ones), codes, None, None, N, K, G)
    assert torch.equal(Y1, Y1[:1].expand(M, N))


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("M", MS)
def test_fused(e0m4, oracle, M, swiglu):
    run_fused(e0m4, oracle, M, 32768, 128, 128, seed=6200 + M, norm=True, swiglu=swiglu, res=True)
