"""Block glue on every tile that carries it: GELU, gate, residual and the row maxima of the output together, on partial tiles of both
edges, with gate rows and scale blocks that end inside a tile, against the CPU oracle."""
import numpy as np
import pytest

import workload
from test_gpu_parity import dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu

TILES = ["w8 dma 64x64 s3 4w", "w8 dma 128x128 a3b2 4w", "w8 dma 128x128 a3b2 4w spread1", "w8 dma 256x192 a3b2 8w spread1",
         "w8 big 256x288", "w8 big 256x256", "w8 big 128x288",
         "f16 dma 64x64 s3 4w", "f16 dma 128x128 a3b2 4w spread1", "f16 dma 256x192 a3b2 8w spread1", "f16 big 256x288", "f16 big 256x256",
         "w4 pipelined 64x64 a3b2 4w any-group", "w4 pipelined 128x128 a3b2 4w any-group", "w4 big 256x288", "w4 big 256x256", "w4 big 128x288"]
# M, K (half as many binary16), N, rows per gate row, rows per scale: one gate row; a gate row that ends inside a 256-row tile and scale
# blocks across every tile boundary; gate rows and scale blocks shorter than a tile; whole 256x288 and 128x288 tiles
SHAPES = [(300, 256, 296, 300, 1), (1152, 384, 600, 384, 96), (513, 256, 1160, 171, 27), (512, 256, 576, 256, 1)]


@pytest.mark.parametrize("M,K,N,gate_rows,R", SHAPES)
@pytest.mark.parametrize("tile", TILES)
def test_glue_on_every_tile(gpu, orc, tile, M, K, N, gate_rows, R):
    import torch
    say(tile, M, K, N, gate_rows, R)
    bits = {"w8": 8, "w4": 4, "f1": 16}[tile[:2]]
    g = workload.rng("tile-glue", M, N)
    residual = (g.standard_normal((M, N), dtype=np.float32) * 2).astype(np.float16)
    gate = g.standard_normal((M // gate_rows, N), dtype=np.float32).astype(np.float16)
    K = K // 2 if bits == 16 else K
    x, bias = workload.activations(M, K, "tile-glue"), workload.bias(N, "tile-glue")
    rowmax = torch.full((M,), 0x7fffffff, dtype=torch.int32, device="cuda")       # the call clears it
    glue = dict(act=gpu.ACT_GELU_TANH, residual=dev(residual), gate=dev(gate), gate_rows=gate_rows, row_absmax=rowmax)
    u_err = 0.0
    if bits == 16:
        w = workload.f16_weights(N, K, "tile-glue")
        x64, w64 = x.astype(np.float64), w.astype(np.float64)
        u = (x64 @ w64.T + bias.astype(np.float64)).astype(np.float32)
        u_err = (K + 1) * 2.0 ** -24 * (np.abs(x64) @ np.abs(w64).T + np.abs(bias.astype(np.float64)))   # fp32 sums in any order
    else:
        lw = workload.layer_weights("tile-glue", K, N, bits, "tile-glue")
        bias = lw["bias"]
        q, s = orc.daq(x, R, nthreads=8)
        u = orc.dequant_w8(orc.gemm_i8(q, lw["w"], nthreads=16), s, R, lw["s_w"], bias) if bits == 8 else \
            orc.dequant_w4(orc.gemm_w4g(q, orc.pack_w4(lw["w"]), 128, nthreads=16), s, R, lw["s_w"], bias)
        w = lw["w"] if bits == 8 else gpu.ql_pack_w4_host(lw["w"])
    gpu.set_gemm_variant(gpu.gemm_variants().index(tile))
    try:
        if bits == 16:
            y = gpu.qlinear_f16(dev(x), dev(w), dev(bias), **glue)
        else:
            y = gpu.qlinear_fused(dev(x), R, dev(w), dev(lw["s_w"]), dev(bias), bits=bits, **glue)
    finally:
        gpu.set_gemm_variant(-1)
    yh = host(y)
    ref = orc.block_glue(u, act=1, residual=residual, gate=gate, gate_rows=gate_rows).astype(np.float64)
    h = orc.block_glue(u, act=1).astype(np.float64)
    # y = fp16(fma(g, fp16(gelu(u)), r)): one fp16 step of h (its GELU is fp32, slope at most 1.13), carried through the gate
    gabs = np.abs(np.repeat(gate.astype(np.float64), gate_rows, 0))
    tol = 1e-3 * np.abs(ref) + gabs * (np.abs(h) * 2.0 ** -10 + 1.13 * u_err) + 2.0 ** -24
    assert (np.abs(yh.astype(np.float64) - ref) <= tol).all()
    assert np.array_equal(host(rowmax).astype(np.uint32), orc.row_absmax_bits(yh))
