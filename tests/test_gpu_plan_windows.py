"""Plans whose layers run several at a time (inputs quantized by one launch, GEMMs together): every output equals that of the layer's own
call, bit for bit, whatever the rows, widths, kinds and the aliasing between outputs and later inputs."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2511_11446_amd as ql
    ql.lib()
    return ql


def _layer(g, K, N, bits, group, bias=True):
    dev = dict(device="cuda", generator=g)
    b = (torch.randn(N, **dev) * 0.02).half() if bias else None
    if bits == 16:
        return dict(K=K, N=N, bits=16, w=(torch.randn(N, K, **dev) * 0.02).half(), w_scale=None, bias=b)
    if bits == 8:
        return dict(K=K, N=N, bits=8, w=torch.randint(-127, 128, (N, K), dtype=torch.int8, **dev), w_scale=torch.rand(N, **dev) * 9e-3 + 1e-3, bias=b)
    return dict(K=K, N=N, bits=4, group=group, w=torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, **dev),
                w_scale=(torch.rand(N, K // group, **dev) * 0.09 + 0.01).half(), bias=b)


def _alone(ql, l, x):
    if l["bits"] == 16:
        return ql.qlinear_f16(x, l["w"], l["bias"])
    if l["bits"] == 8:
        return ql.qlinear_w8a8(x, 1, l["w"], l["w_scale"], l["bias"])
    return ql.qlinear_w4a8(x, 1, l["w"], l["w_scale"], l["bias"], group=l["group"])


# (K, N, bits, group, bias) of each layer
PLANS = {
    "block w8": [(384, 1152, 8, 0, True), (384, 384, 8, 0, False), (384, 1536, 8, 0, True), (1536, 384, 8, 0, True)],
    "all kinds": [(1152, 1000, 4, 288, True), (1152, 264, 16, 0, True), (1152, 640, 4, 128, False), (1152, 392, 8, 0, True),
                  (1152, 130, 4, 32, True), (1152, 200, 4, 64, True), (1152, 648, 4, 192, True), (768, 96, 4, 96, True), (4608, 512, 16, 0, False)],
    "odd inner sizes": [(320, 300, 8, 0, True), (200, 256, 8, 0, True), (256, 136, 16, 0, True), (1032, 128, 8, 0, True), (1028, 64, 8, 0, True)],
    "every row kernel": [(512, 72, 8, 0, True), (1024, 72, 8, 0, True), (1536, 72, 8, 0, True), (2048, 72, 8, 0, True), (3072, 72, 8, 0, True), (4608, 72, 8, 0, True)],
    "short rows": [(128, 136, 8, 0, True), (512, 136, 8, 0, True), (520, 136, 8, 0, True), (1536, 136, 8, 0, True)],
    "wide and narrow": [(4608, 384, 8, 0, True), (384, 513, 8, 0, True), (384, 512, 4, 64, True), (4608, 256, 4, 32, True), (2304, 128, 4, 288, True)],
}


ROWS, ROOM = [129, 512, 1021, 2048], [1, 4]   # ROOM: workspace as a multiple of the recommended one, with more room more layers go together


# (that every kind of tile takes part in a shared GEMM launch here is checked without a GPU, in test_abi_cpu.py)
@pytest.mark.parametrize("M", ROWS)
@pytest.mark.parametrize("name", PLANS)
@pytest.mark.parametrize("room", ROOM)
def test_plan_equals_its_layers(ql, room, name, M):
    g = torch.Generator(device="cuda").manual_seed(M)
    layers = [_layer(g, *s) for s in PLANS[name]]
    x = [torch.randn(M, l["K"], device="cuda", generator=g).half() for l in layers]
    y = [torch.full((M, l["N"]), float("nan"), dtype=torch.float16, device="cuda") for l in layers]
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(room * plan.workspace_bytes(M, 1))
    for _ in range(2):
        plan.run(x, y, M, 1, ws)
    for l, a, b in zip(layers, x, y):
        if l["bits"] == 16:   # fp32 sums in any order, then one rounding to fp16
            exact = a.double() @ l["w"].double().T + (0.0 if l["bias"] is None else l["bias"].double())
            bound = (l["K"] + 1) * 2.0 ** -24 * (a.double().abs() @ l["w"].double().abs().T + 1.0) + exact.abs() * 2.0 ** -11 + 2.0 ** -25
            assert bool(((b.double() - exact).abs() <= bound).all())
        else:
            torch.testing.assert_close(b, _alone(ql, l, a), rtol=0, atol=0)


# Layers whose outputs lie over other layers' inputs and outputs: (buffer, first element) of every input and output.  Layers as in "disjoint" share a GEMM
# launch; which ones still do, and that none does where the order matters, is checked without a GPU, in test_abi_cpu.py
ALIAS_M = 2048
ALIAS_LAYERS = [(384, 1152, 16, 0, True), (384, 1152, 8, 0, True), (384, 1152, 4, 64, True), (384, 1152, 8, 0, True)]
_ROW = 1152
ALIASES = {
    "disjoint": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (6, 0), (7, 0)]),
    "one output": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (4, 0), (4, 0), (4, 0)]),
    "outputs five rows apart": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (5, 5 * _ROW), (7, 0)]),
    "outputs that meet": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (5, ALIAS_M * _ROW), (7, 0)]),
    "an output that a later layer reads": ([(0, 0), (1, 0), (5, 384), (3, 0)], [(4, 0), (5, 0), (6, 0), (7, 0)]),
    "an output over the input of an earlier FP16 layer": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (6, 0), (0, 0)]),
    "an output over the last rows of an FP16 input": ([(0, 3 * _ROW), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (0, ALIAS_M * 384), (7, 0)]),
    "an output over the input of an earlier 8-bit layer": ([(0, 0), (1, 0), (2, 0), (3, 0)], [(4, 0), (5, 0), (1, 0), (7, 0)]),
}


@pytest.mark.parametrize("name", ALIASES)
def test_overlapping_inputs_and_outputs(ql, name):
    M = ALIAS_M
    g = torch.Generator(device="cuda").manual_seed(5)
    layers = [_layer(g, *s) for s in ALIAS_LAYERS]
    t = [torch.randn(2 * M * _ROW, device="cuda", generator=g).half() for _ in range(8)]
    want = [v.clone() for v in t]
    at = lambda bufs, place, width: bufs[place[0]][place[1]: place[1] + M * width].view(M, width)
    xs, ys = ALIASES[name]
    for l, x, y in zip(layers, xs, ys):
        at(want, y, l["N"]).copy_(_alone(ql, l, at(want, x, l["K"]).contiguous()))
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(4 * plan.workspace_bytes(M, 1))
    plan.run([at(t, x, l["K"]) for l, x in zip(layers, xs)], [at(t, y, l["N"]) for l, y in zip(layers, ys)], M, 1, ws)
    for i, (a, b) in enumerate(zip(t, want)):
        # FP16 layers: fp32 sums in any order, then one rounding to fp16
        torch.testing.assert_close(a, b, rtol=2.0 ** -10 if i == ys[0][0] else 0, atol=2.0 ** -14 if i == ys[0][0] else 0)


@pytest.mark.parametrize("bits", [8, 4, 16])
@pytest.mark.parametrize("M,w,room", [(1024, 256, 1), (2048, 512, 7)])
def test_chained_layers_keep_their_order(ql, M, w, room, bits):
    # an output that is the next layer's input, one that is the input of a layer further on, one that overwrites an earlier input, and
    # two layers that write the same output; quantized layers also in place (an FP16 layer reads its input while it writes)
    g = torch.Generator(device="cuda").manual_seed(bits)
    layers = [_layer(g, w, w, b, 64) for b in (8, bits, 4, bits, bits, 8, bits)]
    t = [(torch.randn(M, w, device="cuda", generator=g) * 0.1).half() for _ in range(8)]
    flow = [(0, 1), (1, 2), (3, 4), (1, 5), (5, 3), (0, 6), (6, 7 if bits == 16 else 6)]   # (input, output) of each layer
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(room * plan.workspace_bytes(M, 1))
    want = [v.clone() for v in t]
    for l, (i, o) in zip(layers, flow):
        want[o].copy_(_alone(ql, l, want[i]))
    plan.run([t[i] for i, _ in flow], [t[o] for _, o in flow], M, 1, ws)
    for a, b in zip(t, want):
        if bits == 16:   # an FP16 layer's sums in another order move its output by a rounding, and with it now and then a code of the next layer
            assert float((a.float() - b.float()).norm()) <= 2.0 ** -9 * float(b.float().norm())
        else:
            torch.testing.assert_close(a, b, rtol=0, atol=0, equal_nan=True)


def test_layers_that_write_the_same_output(ql):
    # disjoint inputs, one output for all: the last layer's stays
    M, w = 512, 256
    g = torch.Generator(device="cuda").manual_seed(1)
    layers = [_layer(g, w, w, b, 64) for b in (8, 4, 16, 8)]
    x = [torch.randn(M, w, device="cuda", generator=g).half() for _ in layers]
    y = torch.empty(M, w, dtype=torch.float16, device="cuda")
    plan = ql.Plan(layers, M_max=M)
    plan.run(x, [y] * 4, M, 1, ql.workspace(plan.workspace_bytes(M, 1)))
    torch.testing.assert_close(y, _alone(ql, layers[3], x[3]), rtol=0, atol=0)


def _alone_shared(ql, l, x, R, p_ppm, a_bits):
    if l["bits"] == 16:
        return ql.qlinear_f16(x, l["w"], l["bias"])
    d = ql.daq_quantize_robust(x, R, p_ppm, a_bits) if p_ppm else ql.daq_quantize(x, R)
    if l["bits"] == 8:
        return ql.qgemm_w8a8(d[0], d[1], R, l["w"], l["w_scale"], l["bias"])
    return ql.qgemm_w4a8(d[0], d[1], R, l["w"], l["w_scale"], l["bias"], group=l["group"])


# rows per scale with whole, ragged and many parts per scale block; ranks of the percentile: the maximum, few, many; R = 1 with a percentile;
# more scale blocks than percentiles share launches for
@pytest.mark.parametrize("M,R,p_ppm,a_bits", [(512, 64, 0, 8), (1530, 255, 0, 8), (4096, 1024, 0, 8), (2048, 2048, 0, 8), (1024, 256, 999000, 8),
                                              (518, 74, 990000, 6), (2048, 1024, 999900, 6), (770, 1, 999000, 8), (515, 1, 900000, 4),
                                              (1024, 512, 1000000, 8), (1024, 64, 1, 8),
                                              (8194, 2, 750000, 8)])
@pytest.mark.parametrize("name", ["block w8", "all kinds", "wide and narrow", "every row kernel", "short rows", "odd inner sizes"])
@pytest.mark.parametrize("tight", [False, True])
def test_shared_scales_and_percentiles(ql, name, M, R, p_ppm, a_bits, tight):
    g = torch.Generator(device="cuda").manual_seed(M)
    layers = [l for l in (_layer(g, *s) for s in PLANS[name]) if l["bits"] != 16]
    x = [torch.randn(M, l["K"], device="cuda", generator=g).half() for l in layers]
    x[0][: R + 1] = 0                               # a scale block of zeros, and a row of the next one
    x[-1][:, ::7] *= 30.0
    y = [torch.full((M, l["N"]), float("nan"), dtype=torch.float16, device="cuda") for l in layers]
    plan = ql.Plan(layers, M_max=M)
    need = plan.workspace_bytes(M, R)
    ws = ql.workspace(need if tight else 4 * need)   # with more room more layers go together
    for _ in range(2):
        if p_ppm:
            plan.run_ex(x, y, M, R, ws, p_ppm=p_ppm, a_bits=a_bits)
        else:
            plan.run(x, y, M, R, ws)
    for l, a, b in zip(layers, x, y):
        torch.testing.assert_close(b, _alone_shared(ql, l, a, R, p_ppm, a_bits), rtol=0, atol=0, equal_nan=True)


@pytest.mark.parametrize("p_ppm", [0, 999000])
def test_chained_layers_with_shared_scales(ql, p_ppm):
    M, R, w = 1024, 256, 256
    g = torch.Generator(device="cuda").manual_seed(9)
    layers = [_layer(g, w, w, b, 64) for b in (8, 4, 8, 4, 8)]
    t = [(torch.randn(M, w, device="cuda", generator=g) * 0.1).half() for _ in range(6)]
    flow = [(0, 1), (2, 3), (1, 4), (4, 2), (5, 5)]
    want = [v.clone() for v in t]
    for l, (i, o) in zip(layers, flow):
        want[o].copy_(_alone_shared(ql, l, want[i], R, p_ppm, 8))
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(4 * plan.workspace_bytes(M, R))
    plan.run_ex([t[i] for i, _ in flow], [t[o] for _, o in flow], M, R, ws, p_ppm=p_ppm or None)
    for a, b in zip(t, want):
        torch.testing.assert_close(a, b, rtol=0, atol=0, equal_nan=True)


# so many rows that eight layers together need more threads than a launch holds: one row per scale in the row pass, and a percentile of two rows in
# the selection
@pytest.mark.parametrize("M,R,p_ppm", [(2 ** 23, 1, 0), (2 ** 23 - 4, 1, 0), (2 ** 20, 2, 750000)])
def test_many_rows(ql, M, R, p_ppm):
    g = torch.Generator(device="cuda").manual_seed(7)
    layers = [_layer(g, 8, 8, 8, 0) for _ in range(8)]
    x = torch.randn(M, 8, device="cuda", generator=g).half()
    y = [torch.full((M, 8), float("nan"), dtype=torch.float16, device="cuda") for _ in layers]
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(len(layers) * plan.workspace_bytes(M, R))
    if p_ppm:
        plan.run_ex([x] * 8, y, M, R, ws, p_ppm=p_ppm)
    else:
        plan.run([x] * 8, y, M, R, ws)
    for l, b in zip(layers, y):
        torch.testing.assert_close(b, _alone_shared(ql, l, x, R, p_ppm, 8), rtol=0, atol=0)


# 8-bit layers that are one round of 256x288 tiles together: whole and partial tiles in both directions, one scale for several rows, different inner sizes
ROUND_LAYERS = {
    "block": [(1152, 3456, 8, 0, True), (1152, 1152, 8, 0, True), (1152, 4608, 8, 0, True)],
    "ragged": [(1024, 3016, 8, 0, False), (1152, 4360, 8, 0, True), (640, 1032, 8, 0, True)],
}
ROUNDS = [("block", 2048, 1), ("block", 1793, 1), ("block", 2047, 1), ("block", 2048, 256), ("ragged", 2048, 1), ("ragged", 2001, 1), ("ragged", 1920, 64)]


@pytest.mark.parametrize("name,M,R", ROUNDS)
def test_one_round_of_large_tiles(ql, name, M, R):
    g = torch.Generator(device="cuda").manual_seed(M + R)
    layers = [_layer(g, *s) for s in ROUND_LAYERS[name]]
    x = [torch.randn(M, l["K"], device="cuda", generator=g).half() for l in layers]
    y = [torch.full((M, l["N"]), float("nan"), dtype=torch.float16, device="cuda") for l in layers]
    plan = ql.Plan(layers, M_max=M)
    ws = ql.workspace(4 * plan.workspace_bytes(M, R))
    for _ in range(2):
        plan.run(x, y, M, R, ws)
    for l, a, b in zip(layers, x, y):
        torch.testing.assert_close(b, _alone_shared(ql, l, a, R, 0, 8), rtol=0, atol=0)
