"""Layers that quantize their own rows inside the GEMM, one to five column tiles of 16 to a workgroup, and split K on eight wavefronts, against the CPU
oracle: shapes on both sides of every number of tiles, ragged edges, several rows per scale, gate and residual, groups of every size."""
import numpy as np
import pytest

import workload
from test_gpu_parity import assert_y_close, dev, gpu, host, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


# M, K, N, R: 256 tiles and one row more (1 -> 2 tiles to a workgroup), 2 -> 3, 3 -> 4, 4 (ragged last columns) and one column more, 5 and beyond; all rows of one scale
@pytest.mark.parametrize("M,K,N,R", [(16, 384, 4096, 1), (17, 384, 4096, 1), (250, 1152, 500, 1), (512, 272, 256, 64), (257, 1536, 640, 1), (48, 1152, 4090, 48), (64, 1520, 5113, 1),
                                     (250, 1536, 769, 1), (64, 1520, 4090, 1), (64, 272, 4097, 64),
                                     (256, 1152, 1152, 256), (320, 1152, 1152, 1), (5, 16, 20481, 1)])
def test_w8_tiles_of_a_workgroup(gpu, orc, M, K, N, R):
    say("self-quantizing w8", M, K, N, R)
    x = workload.activations(M, K, "self-q")
    lw = dict(w=workload.w8_codes(N, K, "self-q"), s_w=workload.w8_scales(N, "self-q"), bias=workload.bias(N, "self-q"))
    ref = orc.qlinear_w8a8(x, R, lw["w"], lw["s_w"], lw["bias"], want_debug=False)["y"]
    assert assert_y_close(host(gpu.qlinear_w8a8(dev(x), R, dev(lw["w"]), dev(lw["s_w"]), dev(lw["bias"]))), ref) == 0


# groups that leave wavefronts without one, several to a wavefront, several rounds; K beyond what a workgroup quantizes: eight wavefronts on 16x16, two
# 16x16 and 32x32 tiles
@pytest.mark.parametrize("M,K,N,group", [(16, 384, 100, 128), (40, 1152, 1152, 288), (128, 1152, 1152, 128), (64, 1536, 1530, 32), (250, 768, 768, 192), (200, 384, 1100, 32),
                                         (250, 1536, 1000, 128), (60, 768, 4090, 96), (16, 4608, 700, 128), (70, 4608, 1100, 288), (130, 4608, 1152, 64), (100, 2304, 500, 1152)])
def test_w4_tiles_of_a_workgroup(gpu, orc, M, K, N, group):
    say("self-quantizing w4", M, K, N, group)
    g = workload.rng("self-q4", M, N)
    x, codes, sw, bias = workload.activations(M, K, "self-q4"), workload.w4_codes(N, K, "self-q4"), workload.w4_scales_group(N, K, group, "self-q4"), workload.bias(N, "self-q4")
    residual, gate = (g.standard_normal(s, dtype=np.float32).astype(np.float16) for s in ((M, N), (1, N)))
    q, s = orc.daq(x, 1)
    u = orc.dequant_w4(orc.gemm_w4g(q, orc.pack_w4(codes), group, nthreads=16), s, 1, sw, bias)
    w4, sd, bd = dev(gpu.ql_pack_w4_host(codes)), dev(sw), dev(bias)
    assert np.array_equal(host(gpu.qlinear_w4a8(dev(x), 1, w4, sd, bd, group=group)).view(np.uint16), orc.block_glue(u).view(np.uint16))
    y = gpu.qlinear_fused(dev(x), 1, w4, sd, bd, bits=4, group=group, residual=dev(residual), gate=dev(gate), gate_rows=M)
    assert np.array_equal(host(y).view(np.uint16), orc.block_glue(u, residual=residual, gate=gate, gate_rows=M).view(np.uint16))


def test_outputs_over_the_inputs_of_a_wide_layer(gpu):
    """Several column tiles to a workgroup, outputs over the inputs that other workgroups still read: two launches."""
    import torch
    M = K = 384
    x, lw = workload.activations(M, K, "self-place"), workload.layer_weights("self-place", K, K, 8, "self-place")
    args = (dev(lw["w"]), dev(lw["s_w"]), dev(lw["bias"]))
    apart, xd = gpu.qlinear_w8a8(dev(x), 1, *args), dev(x)
    gpu.qlinear_w8a8(xd, 1, *args, y=xd)
    assert torch.equal(apart, xd)
