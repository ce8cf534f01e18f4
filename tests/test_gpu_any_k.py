"""The DMA tiles for rows that are no whole K steps: every way in which the last step of 128 bytes can be cut short, operands that start at
any word, partial tiles with gate and residual, against the CPU oracle."""
import numpy as np
import pytest

import workload
from test_gpu_parity import _f16_tolerance, assert_y_close, dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu

TILES = ["dma any-K 64x64 s3 4w", "dma any-K 128x128 a3b2 4w spread1"]


def _forced(gpu, tile, call):
    gpu.set_gemm_variant(gpu.gemm_variants().index(tile))
    try:
        return call()
    finally:
        gpu.set_gemm_variant(-1)


# one piece; a second one of 4 bytes; a step less a word, whole, and a word more; two and three steps (as many as the rings hold) and behind them
@pytest.mark.parametrize("M,K,N", [(65, 16, 33), (40, 20, 64), (130, 124, 70), (64, 128, 129), (129, 132, 40), (70, 256, 130), (33, 260, 65), (200, 372, 72), (140, 508, 200),
                                   (300, 1160, 136)])
@pytest.mark.parametrize("tile", TILES)
def test_w8_last_step(gpu, orc, tile, M, K, N):
    import torch
    say(tile, M, K, N)
    x = workload.activations(M, K, "any-k")
    lw = dict(w=workload.w8_codes(N, K, "any-k"), s_w=workload.w8_scales(N, "any-k"), bias=workload.bias(N, "any-k"))
    ref = orc.qlinear_w8a8(x, 1, lw["w"], lw["s_w"], lw["bias"], want_debug=False)["y"]
    buf = torch.zeros(N * K + 4, dtype=torch.int8, device="cuda")
    view = buf[4:].view(N, K)
    view.copy_(dev(lw["w"]))
    for w in (dev(lw["w"]), view):
        y = _forced(gpu, "w8 " + tile, lambda: gpu.qlinear_w8a8(dev(x), 1, w, dev(lw["s_w"]), dev(lw["bias"])))
        assert assert_y_close(host(y), ref) == 0


@pytest.mark.parametrize("M,K,N", [(65, 8, 33), (40, 10, 64), (130, 62, 70), (129, 66, 40), (33, 130, 65), (140, 254, 200), (300, 580, 136)])
@pytest.mark.parametrize("tile", TILES)
def test_f16_last_step(gpu, orc, tile, M, K, N):
    """What pads the last step is not multiplied with infinities or NaN of either operand."""
    say(tile, M, K, N)
    g = workload.rng("any-k16", M, K, N)
    x = workload.activations(M, K, "any-k16")
    w = (g.standard_normal((N, K), dtype=np.float32) * 0.05).astype(np.float16)
    x[x == 0] = 1
    w[w == 0] = 0.05
    w[0, K - 1], w[N // 2, max(K - 8, 0)], w[N - 1, 0] = np.inf, -np.inf, np.nan
    x[M // 2, K - 2] = np.inf
    y, ref = host(_forced(gpu, "f16 " + tile, lambda: gpu.qlinear_f16(dev(x), dev(w), None))), orc.linear_f16(x, w, None, nthreads=16)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
    rows, cols = np.arange(M) != M // 2, ~np.isin(np.arange(N), [0, N // 2, N - 1])
    y, ref = y[np.ix_(rows, cols)], ref[np.ix_(rows, cols)]
    assert (np.abs(y.astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(x[rows], w[cols], ref)).all()
