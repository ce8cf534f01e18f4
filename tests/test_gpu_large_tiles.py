"""The large-tile GEMM on every one of its tiles, against the CPU oracle: partial tiles on both edges, the shortest K, even and
odd numbers of K steps, several tiles per workgroup with and without partial ones among them, and block glue in the epilogue."""
import numpy as np
import pytest

import workload
from test_gpu_parity import _f16_tolerance, assert_y_close, dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu

TILES = ["w8 big 256x288", "w8 big 256x256", "w8 big 128x288", "f16 big 256x288", "f16 big 256x256"]
# M, K (8-bit codes; half as many binary16), N
SHAPES = [(1, 256, 8), (300, 256, 296), (513, 384, 1160), (16384, 384, 2304), (17000, 256, 2056)]


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("tile", TILES)
def test_large_tiles(gpu, orc, tile, M, K, N):
    say(tile, M, K, N)
    g = workload.rng("large", M, N)
    rows = np.arange(M) if M <= 600 else np.unique(np.concatenate([g.choice(M, size=400, replace=False), np.arange(M - 60, M)]))
    gate_rows = max(d for d in range(1, 129) if M % d == 0)
    res = g.standard_normal((M, N), dtype=np.float32).astype(np.float16)
    gate = g.standard_normal((M // gate_rows, N), dtype=np.float32).astype(np.float16)
    f16 = tile.startswith("f16")
    if f16:
        K //= 2
    x = workload.activations(M, K, "large")
    lw = workload.layer_weights("large", K, N, 8, "large") if not f16 else None
    w = (g.standard_normal((N, K), dtype=np.float32) * 0.05).astype(np.float16) if f16 else lw["w"]
    bias = workload.bias(N, "large")
    xd, wd, glue = dev(x), dev(w), dict(residual=dev(res), gate=dev(gate), gate_rows=gate_rows)
    gpu.set_gemm_variant(gpu.gemm_variants().index(tile))
    try:
        if f16:
            ys = [gpu.qlinear_f16(xd, wd, dev(bias)), gpu.qlinear_f16(xd, wd, None, **glue)]
        else:
            q, s = gpu.daq_quantize(xd, 1)
            ys = [gpu.qgemm_w8a8(q, s, 1, wd, dev(lw["s_w"]), dev(bias)), gpu.qgemm_w8a8(q, s, 1, wd, dev(lw["s_w"]), None),
                  gpu.qlinear_fused(xd, 1, wd, dev(lw["s_w"]), dev(bias), bits=8, **glue)]
    finally:
        gpu.set_gemm_variant(-1)
    ys = [host(y)[rows] for y in ys]
    if f16:
        ref = orc.linear_f16(x[rows], w, bias, nthreads=16)
        assert (np.abs(ys[0].astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(x[rows], w, ref)).all()
        h = orc.linear_f16(x[rows], w, None, nthreads=16)
        gr = gate[rows // gate_rows].astype(np.float32)
        ref = (gr * h.astype(np.float32) + res[rows].astype(np.float32)).astype(np.float16)
        # h may sit one fp16 ulp from the oracle's (fp32 against fp64 sums); the gate carries that into y
        tol = _f16_tolerance(x[rows], w, h) * np.abs(gr) + 2.0 ** -10 * np.abs(ref.astype(np.float64)) + 2.0 ** -24
        assert (np.abs(ys[1].astype(np.float64) - ref.astype(np.float64)) <= tol).all()
        return
    q, s = orc.daq(x[rows], 1, nthreads=16)
    acc = orc.gemm_i8(q, w, nthreads=16)
    assert assert_y_close(ys[0], orc.epilogue_w8(acc, s, 1, lw["s_w"], bias)) == 0
    assert assert_y_close(ys[1], orc.epilogue_w8(acc, s, 1, lw["s_w"], None)) == 0
    u = orc.dequant_w8(acc, s, 1, lw["s_w"], bias)
    ref = np.concatenate([orc.block_glue(u[i:i + 1], act=0, residual=res[r:r + 1], gate=gate[r // gate_rows:r // gate_rows + 1], gate_rows=1) for i, r in enumerate(rows)])
    assert assert_y_close(ys[2], ref) == 0


@pytest.mark.parametrize("tile", ["f16 big 256x288", "f16 big 256x256", "f16 dma 128x128 a3b2 4w spread1"])
def test_binary16_operand_above_two_gigabytes(gpu, orc, tile):
    """2^20 rows of 2176 bytes: the last rows start at byte offsets that only an unsigned 32-bit number holds."""
    import torch
    M, K, N = 1 << 20, 1088, 256
    say(tile, M, K, N)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.empty((M, K), dtype=torch.float16, device="cuda").normal_(generator=g)
    w = torch.empty((N, K), dtype=torch.float16, device="cuda").normal_(0.0, 0.05, generator=g)
    assert x.numel() * 2 > 2 ** 31
    gpu.set_gemm_variant(gpu.gemm_variants().index(tile))
    try:
        y = gpu.qlinear_f16(x, w, None)
    finally:
        gpu.set_gemm_variant(-1)
    edge = 2 ** 31 // (2 * K)
    rows = torch.tensor([0, 1, 777777, *range(edge - 20, edge + 20), *range(M - 40, M)], device="cuda")
    xs, ys = host(x[rows]), host(y[rows])
    ref = orc.linear_f16(xs, host(w), None, nthreads=16)
    assert (np.abs(ys.astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(xs, host(w), ref)).all()
