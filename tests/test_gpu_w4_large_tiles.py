"""The large-tile 4-bit GEMM (groups of 128) on every one of its tiles, against the CPU oracle: partial tiles on both edges, the shortest
K and the most groups, odd and even numbers of groups, several tiles per workgroup with and without partial ones among them, and
block glue in the epilogue."""
import numpy as np
import pytest

import workload
from test_gpu_parity import assert_y_close, dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu

TILES = ["w4 big 256x288", "w4 big 256x256", "w4 big 128x288"]
SHAPES = [(1, 256, 8), (300, 256, 296), (513, 384, 1160), (130, 5120, 568), (16384, 384, 2304), (17000, 256, 2056)]


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("tile", TILES)
def test_w4_large_tiles(gpu, orc, tile, M, K, N):
    say(tile, M, K, N)
    g = workload.rng("w4 large", M, N)
    rows = np.arange(M) if M <= 600 else np.unique(np.concatenate([g.choice(M, size=300, replace=False), np.arange(M - 60, M)]))
    gate_rows = max(d for d in range(1, 129) if M % d == 0)
    res = g.standard_normal((M, N), dtype=np.float32).astype(np.float16)
    gate = g.standard_normal((M // gate_rows, N), dtype=np.float32).astype(np.float16)
    x = workload.activations(M, K, "w4 large")
    lw = workload.layer_weights("w4 large", K, N, 4, "w4 large")
    w, sw, bias = lw["w"].copy(), lw["s_w"], lw["bias"]
    w[::3] = np.where(w[::3] >= 0, 7, -8)   # the largest partial sums
    w4 = orc.pack_w4(w)
    xd, wd, sd = dev(x), dev(w4), dev(sw)
    q, s = gpu.daq_quantize(xd, 1)
    gpu.set_gemm_variant(gpu.gemm_variants().index(tile))
    try:
        ys = [gpu.qgemm_w4a8(q, s, 1, wd, sd, dev(bias)), gpu.qgemm_w4a8(q, s, 1, wd, sd, None),
              gpu.qlinear_fused(xd, 1, wd, sd, dev(bias), bits=4, residual=dev(res), gate=dev(gate), gate_rows=gate_rows)]
    finally:
        gpu.set_gemm_variant(-1)
    ys = [host(y)[rows] for y in ys]
    q, s = orc.daq(x[rows], 1, nthreads=16)
    P = orc.gemm_w4g(q, w4, 128, nthreads=16)
    assert assert_y_close(ys[0], orc.epilogue_w4(P, s, 1, sw, bias)) == 0
    assert assert_y_close(ys[1], orc.epilogue_w4(P, s, 1, sw, None)) == 0
    u = orc.dequant_w4(P, s, 1, sw, bias)
    ref = np.concatenate([orc.block_glue(u[i:i + 1], act=0, residual=res[r:r + 1], gate=gate[r // gate_rows:r // gate_rows + 1], gate_rows=1) for i, r in enumerate(rows)])
    assert assert_y_close(ys[2], ref) == 0
