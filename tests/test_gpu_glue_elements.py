"""Gate and residual where they meet the outputs one by one, against the CPU oracle."""
import numpy as np
import pytest

import workload
from test_gpu_parity import dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


# partial tiles of both edges (the last ones with blocks wholly behind the edge), whole tiles of an odd width, outputs that no 16-byte piece reaches, gate rows that end inside a tile; split-K, the register-staged kernel and the DMA tiles
@pytest.mark.parametrize("tile,M,K,N,gate_rows", [(None, 35, 48, 33, 7), (None, 300, 136, 2050, 60), ("w8 edge any-K", 200, 136, 101, 40),
                                                  ("w8 dma 64x64 s3 4w", 300, 256, 301, 300), ("w8 dma 128x128 a3b2 4w spread1", 300, 256, 301, 50),
                                                  ("w8 dma 256x192 a3b2 8w spread1", 259, 256, 389, 37), ("w8 edge any-K", 2912, 24, 2890, 56)])
def test_w8_gate_and_residual_element_by_element(gpu, orc, tile, M, K, N, gate_rows):
    say(tile, M, K, N, gate_rows)
    g = workload.rng("elements", M, N)
    x = workload.activations(M, K, "elements")
    residual, gate = (g.standard_normal(s, dtype=np.float32).astype(np.float16) for s in ((M, N), (M // gate_rows, N)))
    lw = dict(w=workload.w8_codes(N, K, "elements"), s_w=workload.w8_scales(N, "elements"), bias=workload.bias(N, "elements"))
    q, s = orc.daq(x, 1)
    ref = orc.block_glue(orc.dequant_w8(orc.gemm_i8(q, lw["w"], nthreads=8), s, 1, lw["s_w"], lw["bias"]), residual=residual, gate=gate, gate_rows=gate_rows)
    call = lambda **kw: gpu.qlinear_fused(dev(x), 1, dev(lw["w"]), dev(lw["s_w"]), dev(lw["bias"]), gate=dev(gate), gate_rows=gate_rows, **kw)
    r = dev(residual)
    for kw in (dict(residual=r), dict(residual=r, y=r)):       # the second in place
        gpu.set_gemm_variant(-1 if tile is None else gpu.gemm_variants().index(tile))
        try:
            y = call(**kw)
        finally:
            gpu.set_gemm_variant(-1)
        assert np.array_equal(host(y).view(np.uint16), ref.view(np.uint16))
