"""Prompts whose last row tile of 128 holds 64 rows or fewer: those tiles are computed in two blocks of 32 rows and numbered behind
the whole ones (32776 and, gated, 32768 columns: as many tiles as compute units; 11016 with six row tiles likewise; 200: too
few for that)."""
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
    plain(e0m4, oracle, M, N, K, fmt, G)


# more than one round of the K loop on two row blocks: two, three and five pairs of K slices
@pytest.mark.parametrize("fmt,G", [("e0m4", 64), ("e0m4", 128), ("e0m8", 128), ("bf16", 128)])
@pytest.mark.parametrize("M,K", [(129, 256), (300, 384), (192, 640)])
def test_longer_rows(e0m4, oracle, M, K, fmt, G):
    plain(e0m4, oracle, M, 32776, K, fmt, G)


# six row tiles, of which five, the whole ones, are more than a panel of four: both numberings, and the same bits without panels
@pytest.mark.parametrize("fmt,G", [("e0m4", 128), ("bf16", 128)])
@pytest.mark.parametrize("M", [641, 700])
def test_panels(e0m4, oracle, M, fmt, G):
    Y = plain(e0m4, oracle, M, 11016, 256, fmt, G)
    e0m4.e0m4_set_knob("gemm_panel", -1)
    try:
        Y2 = plain(e0m4, oracle, M, 11016, 256, fmt, G)
    finally:
        e0m4.e0m4_set_knob("gemm_panel", 0)
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))


def plain(e0m4, oracle, M, N, K, fmt, G):
    if fmt == "bf16":
        codes, What, _ = assert_bf16_quantize_exact(e0m4, oracle, synth_inputs.weights_bf16(N, K, seed=6000 + N), G)
        X = synth_inputs.activations_bf16(M, K, seed=6100 + M)
        Yref, absdot = oracle.bf16_matmul(X, What)
        Y = e0m4.e0m4_bf16_matmul(bf_dev(X), codes, N, K, G)
        check_bf16_matmul(oracle, Y, Yref, absdot, "bf16 M=%d" % M)
        return Y
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
    return Y


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("M,K", [(129, 128), (192, 128), (300, 128), (300, 640)])
def test_fused(e0m4, oracle, M, K, swiglu):
    run_fused(e0m4, oracle, M, 32768, K, 128, seed=6200 + M, norm=True, swiglu=swiglu, res=True)
