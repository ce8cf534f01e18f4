"""Layers of few rows and of inner sizes that no K step divides: the split-K kernel (with and without the quantization inside
the GEMM), the register-staged kernel (forced, and for odd rows and alignments, which nothing else takes) and the 64x64 tiles of the pipelined kernels, at the
edges of their tiles, steps, rounds and alignments, against the CPU oracle."""
import numpy as np
import pytest

import workload
from test_gpu_parity import _f16_tolerance, assert_y_close, dev, gpu, host, run_w8, say  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


# M, K, N, R
W8 = [(1, 16, 1, 1), (15, 48, 33, 1), (17, 144, 16, 1), (31, 1536, 31, 1), (33, 1552, 65, 1),   # 16x16 tiles; quantization inside up to K = 1536
      (64, 1152, 96, 64), (96, 576, 48, 32),            # several rows per scale: partial maxima, then one launch
      (100, 4608, 700, 1), (330, 2320, 1160, 1),        # 32x32 tiles, two rounds of them
      (500, 2432, 1152, 1), (3000, 256, 4090, 1),       # more 32x32 tiles than one round, 256x192 tiles just beyond one: other tiles
      (2300, 64, 2176, 1), (2177, 448, 2048, 7), (17000, 2112, 520, 17000),                      # an odd multiple of 64, more than 256 tiles
      (130, 1160, 70, 1), (130, 1157, 70, 1), (3, 7, 5, 1), (2100, 136, 1100, 1)]   # rows that end on whole words (DMA tiles) and on bytes (register-staged)


@pytest.mark.parametrize("M,K,N,R", W8)
def test_w8_small_and_ragged(gpu, orc, M, K, N, R):
    say("w8 small", M, K, N, R)
    run_w8(gpu, orc, M, K, N, R, ("small", M, K, N), use_bias=(M % 2 == 0), check_exact=True)


# rows that end on 16, 8, 4 and 2 bytes and on one; 64x64 tiles and, from 512 of them on, 128x128 ones
EDGE = [(130, 1168, 70), (130, 1160, 70), (130, 1156, 70), (130, 1154, 70), (130, 1157, 70), (2100, 136, 1100), (2900, 141, 2870)]


@pytest.mark.parametrize("M,K,N", EDGE)
def test_w8_register_staged(gpu, orc, M, K, N):
    say("w8 staged", M, K, N)
    gpu.set_gemm_variant(gpu.gemm_variants().index("w8 edge any-K"))
    try:
        run_w8(gpu, orc, M, K, N, 1, ("staged", M, K, N), use_bias=(M % 4 == 0), check_exact=True)
    finally:
        gpu.set_gemm_variant(-1)


@pytest.mark.parametrize("M,K,N", EDGE + [(700, 136, 700), (130, 1151, 70)])
def test_f16_register_staged(gpu, orc, M, K, N):
    """With infinities and NaN in the last inputs of a row: what pads the last K step is not multiplied with them."""
    say("f16 staged", M, K, N)
    g = workload.rng("staged16", M, K, N)
    x = workload.activations(M, K, "staged16")
    w = (g.standard_normal((N, K), dtype=np.float32) * 0.05).astype(np.float16)
    x[x == 0] = 1
    w[w == 0] = 0.05
    w[0, K - 1], w[N // 2, K - 8], w[N - 1, K - 3] = np.inf, -np.inf, np.nan
    x[M // 2, K - 2] = np.inf
    gpu.set_gemm_variant(gpu.gemm_variants().index("f16 edge any-K"))
    try:
        y = host(gpu.qlinear_f16(dev(x), dev(w), None))
    finally:
        gpu.set_gemm_variant(-1)
    ref = orc.linear_f16(x, w, None, nthreads=16)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
    rows, cols = np.arange(M) != M // 2, ~np.isin(np.arange(N), [0, N // 2, N - 1])
    y, ref = y[np.ix_(rows, cols)], ref[np.ix_(rows, cols)]
    assert (np.abs(y.astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(x[rows], w[cols], ref)).all()


@pytest.mark.parametrize("offset", [1, 2, 8])
def test_w8_misaligned_operands(gpu, orc, offset):
    """Weights that start `offset` bytes off a 16-byte boundary: the DMA kernels must step aside."""
    import torch
    M, K, N = 70, 256, 40
    say("w8 misaligned", offset)
    x = workload.activations(M, K, "mis")
    lw = workload.layer_weights("mis", K, N, 8, "mis")
    ref = orc.qlinear_w8a8(x, 1, lw["w"], lw["s_w"], lw["bias"], want_debug=False)["y"]
    buf = torch.zeros(N * K + 16, dtype=torch.int8, device="cuda")
    view = buf[offset:offset + N * K].view(N, K)
    view.copy_(dev(lw["w"]))
    y = gpu.qlinear_w8a8(dev(x), 1, view, dev(lw["s_w"]), dev(lw["bias"]))
    assert assert_y_close(host(y), ref) == 0


# M, K, N, group: odd numbers of 32-wide slices, one and several rounds of groups, 64x64 tiles with ragged edges
W4 = [(1, 32, 1, 32), (17, 288, 33, 288), (16, 96, 16, 96), (5, 4608, 17, 32), (40, 4608, 100, 64), (33, 1184, 40, 32), (70, 1184, 40, 32),
      (200, 1152, 1160, 192), (520, 1152, 1160, 288), (321, 4608, 193, 32), (2100, 160, 40, 32)]


@pytest.mark.parametrize("M,K,N,group", W4)
def test_w4_small_and_ragged(gpu, orc, M, K, N, group):
    say("w4 small", M, K, N, group)
    x = workload.activations(M, K, "small4", group)
    lw = workload.layer_weights("small4", K, N, 4, group) if K % 128 == 0 else dict(w=workload.w4_codes(N, K, "small4"), bias=workload.bias(N, "small4"))
    sw = workload.w4_scales_group(N, K, group, "small4")
    q, s = orc.daq(x, 1)
    P = orc.gemm_w4g(q, orc.pack_w4(lw["w"]), group, nthreads=8)
    ref = orc.epilogue_w4(P, s, 1, sw, lw["bias"])
    w4 = dev(gpu.ql_pack_w4_host(lw["w"]))
    out = gpu.qlinear_w4a8(dev(x), 1, w4, dev(sw), dev(lw["bias"]), debug=True, group=group)
    assert np.array_equal(host(out["P"]), P)
    assert assert_y_close(host(out["y"]), ref) == 0
    y = gpu.qlinear_w4a8(dev(x), 1, w4, dev(sw), dev(lw["bias"]), group=group)      # few rows: quantized inside the GEMM
    assert assert_y_close(host(y), ref) == 0


@pytest.mark.parametrize("M,K,N,R,group,storage", [(64, 384, 40, 32, 32, 8), (192, 384, 300, 64, 96, 8), (1024, 384, 600, 64, 128, 4), (96, 96, 24, 24, 32, 8),
                                                   (256, 4608, 1100, 128, 64, 8)])
def test_channel_group_scales_by_block_size(gpu, orc, M, K, N, R, group, storage):
    say("channel groups", M, K, N, R, group, storage)
    g = workload.rng("small-cg", M, K, N)
    x = workload.activations(M, K, "small-cg", sigma=0.8)
    codes = g.integers(-8, 8, (N, K), dtype=np.int8)
    s_w, bias = workload.w4_scales_group(N, K, group, "small-cg"), workload.bias(N, "small-cg")
    q, a = orc.daq_cg(x, R, group, nthreads=8)
    ref = orc.epilogue_cg(orc.gemm_i8g(q, codes, group, nthreads=16), a, R, s_w, bias)
    w = dev(gpu.ql_pack_w4_host(codes)) if storage == 4 else dev(codes)
    y = gpu.qlinear_grouped(dev(x), R, w, dev(s_w), group, dev(bias), act_group=group, storage=storage)
    assert assert_y_close(host(y), ref) == 0


@pytest.mark.parametrize("M,K,N", [(1, 8, 1), (17, 24, 33), (40, 1160, 100), (130, 1154, 70), (500, 4608, 1152), (3000, 192, 4090)])
def test_f16_small_and_ragged(gpu, orc, M, K, N):
    say("f16 small", M, K, N)
    g = workload.rng("small16", M, K, N)
    x = workload.activations(M, K, "small16")
    w = (g.standard_normal((N, K), dtype=np.float32) * 0.05).astype(np.float16)
    b = workload.bias(N, "small16")
    ref = orc.linear_f16(x, w, b, nthreads=16)
    y = host(gpu.qlinear_f16(dev(x), dev(w), dev(b)))
    assert (np.abs(y.astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(x, w, ref)).all()


# 17 and 256 slabs per scale block (merged by the workgroup together), 16 (each thread for itself); one, two and three rows side by side;
# the last shape of the row kernels and the first one of the slabs behind it
@pytest.mark.parametrize("M,K,R,cg", [(544, 2568, 272, 24), (4096, 384, 4096, 96), (512, 1160, 256, 8), (1024, 4096, 1024, 32), (2048, 4608, 64, 288), (2112, 4608, 64, 288)])
def test_channel_group_slabs(gpu, orc, M, K, R, cg):
    say("channel-group slabs", M, K, R, cg)
    x = workload.activations(M, K, "slabs", R, cg)
    q_ref, a_ref = orc.daq_cg(x, R, cg, nthreads=16)
    q, a = gpu.daq_quantize_cg(dev(x), R, cg)
    assert np.array_equal(host(a).view(np.uint32), a_ref.view(np.uint32)) and np.array_equal(host(q), q_ref)


# 16x16 and 32x32 split-K tiles with one to seven chunks of the last K step missing, the DMA tiles
@pytest.mark.parametrize("M,K,N", [(40, 1160, 100), (17, 24, 33), (5, 120, 16), (500, 4616, 500), (700, 136, 700), (130, 1154, 70), (96, 256, 2048)])
def test_f16_infinite_operands(gpu, orc, M, K, N):
    """Infinities and NaN in the last inputs of a row reach the outputs that they belong to and no others: what pads a row's last K
    step must not be multiplied with them."""
    say("f16 infinities", M, K, N)
    g = workload.rng("inf16", M, K, N)
    x = workload.activations(M, K, "inf16")
    w = (g.standard_normal((N, K), dtype=np.float32) * 0.05).astype(np.float16)
    x[x == 0] = 1
    w[w == 0] = 0.05
    w[0, K - 1], w[N // 2, K - 8], w[N - 1, K - 3] = np.inf, -np.inf, np.nan
    x[M // 2, K - 2] = np.inf
    y, ref = host(gpu.qlinear_f16(dev(x), dev(w), None)), orc.linear_f16(x, w, None, nthreads=16)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
    rows, cols = np.arange(M) != M // 2, ~np.isin(np.arange(N), [0, N // 2, N - 1])
    y, ref = y[np.ix_(rows, cols)], ref[np.ix_(rows, cols)]
    assert (np.abs(y.astype(np.float64) - ref.astype(np.float64)) <= _f16_tolerance(x[rows], w[cols], ref)).all()


@pytest.mark.parametrize("M,bits,R", [(16, 8, 1), (40, 4, 1), (64, 8, 64)])
def test_outputs_over_the_inputs(gpu, M, bits, R):
    """A square layer whose outputs replace its inputs: no workgroup may still read what another one has overwritten."""
    import torch
    K = 384
    say("in place", M, bits, R)
    x = workload.activations(M, K, "in-place")
    lw = workload.layer_weights("in-place", K, K, bits, "in-place")
    w = dev(lw["w"] if bits == 8 else gpu.ql_pack_w4_host(lw["w"]))
    layer = gpu.qlinear_w8a8 if bits == 8 else gpu.qlinear_w4a8
    apart = layer(dev(x), R, w, dev(lw["s_w"]), dev(lw["bias"]))
    xd = dev(x)
    assert layer(xd, R, w, dev(lw["s_w"]), dev(lw["bias"]), y=xd).data_ptr() == xd.data_ptr()
    assert torch.equal(apart, xd)


def _aligned(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("M,K,R", [(256, 1152, 64), (24, 96, 8), (512, 4608, 256)])
def test_smaller_workspaces(gpu, M, K, R):
    """One set of histogram words per scale block (386 of them, and one word for tau), or one word per channel-group scale, is still
    enough: the kernels that need more step aside."""
    import torch
    say("smaller workspaces", M, K, R)
    x = dev(workload.activations(M, K, "less"))
    nblk, group = M // R, 32
    small = gpu.workspace(_aligned(4 * nblk) + _aligned(4 * 386 * nblk))
    want, got = gpu.daq_quantize_robust(x, R, 990000, 6), gpu.daq_quantize_robust(x, R, 990000, 6, ws=small)
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
    q, s = gpu.daq_quantize_cg(x, R, group)
    q2, s2, ws = torch.zeros_like(q), torch.zeros_like(s), gpu.workspace(_aligned(4 * nblk * (K // group)))
    assert gpu.lib().daq_quantize_cg(x.data_ptr(), M, K, R, group, q2.data_ptr(), s2.data_ptr(), ws.data_ptr(), ws.numel(), None) == 0
    assert torch.equal(q, q2) and torch.equal(s, s2)


def test_plan_on_the_workspace_of_its_widest_layer(gpu):
    """A plan's layer of K = 8192 on a workspace sized for K = 8193 alone, which has no room for its partial maxima: the atomic
    maxima step in, nothing behind the workspace is written, and the codes are those of a workspace with room."""
    import torch
    M, N, R = 8192, 24, 8192
    say("plan workspace", M, R)
    layers = [dict(K=K, N=N, bits=8, w=dev(workload.w8_codes(N, K, "plan-ws")), w_scale=dev(workload.w8_scales(N, "plan-ws")), bias=None) for K in (8193, 8192)]
    xs = [dev(workload.activations(M, l["K"], "plan-ws")) for l in layers]
    small = _aligned(M * 8193) + _aligned(4) + _aligned(4) + _aligned(4 * 386)
    plan = gpu.Plan(layers, M_max=M)
    assert plan.workspace_bytes(M, R) > small
    whole, room = gpu.workspace(small + (1 << 16)), gpu.workspace(plan.workspace_bytes(M, R))
    whole.fill_(0x5a)
    got, want = ([torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in layers] for _ in range(2))
    plan.run(xs, got, M, R, whole[:small])
    plan.run(xs, want, M, R, room)
    assert bool((whole[small:] == 0x5a).all()) and all(torch.equal(a, b) for a, b in zip(got, want))
