"""Cases by which the speed of the quantized linear path is judged: what they are, their inputs, one pass, the work in it.

A case is one of four kinds of call that a program makes of this package:

  layer    one linear layer: DAQ + INT8 GEMM + dequantization (8- or 4-bit weights) or the FP16 layer, optionally with
           GELU or a gated residual in its epilogue
  plan     the linears of one or more transformer blocks under a per-layer bit plan, through Plan.run / Plan.run_ex
  block    one block as an adaptive-LayerNorm transformer runs it: LayerNorm + modulation + DAQ, qkv, the projection and
           the MLP with GELU and gated residuals in the epilogues
  grouped  one layer with group scales of any code width, and activation scales per image and channel group

A block of width w has the layers qkv (w -> 3w), proj (w -> w), fc1 (w -> 4w) and fc2 (4w -> w).
"""
import math

import torch

import paper_2511_11446_amd as ql
import workload

WIDTHS = (384, 768, 1024, 1152)
W4_GROUPS = (32, 64, 128, 192, 288)


def listed():
    return [
        # one linear of one 256-token image, one activation scale for the tensor: the smallest call of a sampling loop
        dict(name="layer_w8_m256_tensor", kind="layer", M=256, K=1152, N=1152, bits=8, group=0, R=256, act=0, gated=False),
        # the same end of the range with 4-bit weights and a long K: a few tokens through the MLP's output layer
        dict(name="layer_w4_m64_long_k", kind="layer", M=64, K=4608, N=1152, bits=4, group=128, R=1, act=0, gated=False),
        # nothing divides a tile: rows, inputs and outputs of a layer that is not a transformer's own
        dict(name="layer_w8_ragged", kind="layer", M=1021, K=1160, N=1000, bits=8, group=0, R=1, act=0, gated=False),
        # a layer the plan leaves in FP16, with the MLP's GELU
        dict(name="layer_f16_gelu_m2048", kind="layer", M=2048, K=1152, N=4608, bits=16, group=0, R=1, act=1, gated=False),
        # 8-bit block, 8 images of 256 tokens, one scale per token
        dict(name="plan_w8_m2048", kind="plan", M=2048, width=1152, blocks=1, plan="w8", R=1, p_ppm=0, a_bits=8),
        # attention layers 8-bit, MLP layers 4-bit, 32 images
        dict(name="plan_mixed_m8192", kind="plan", M=8192, width=1152, blocks=1, plan="mixed", R=1, p_ppm=0, a_bits=8),
        # 8-bit block at the 512-pixel size: 16 images of 1024 tokens
        dict(name="plan_w8_m16384", kind="plan", M=16384, width=1152, blocks=1, plan="w8", R=1, p_ppm=0, a_bits=8),
        # scales as the method's formula prints them: 99.9th percentile of each image
        dict(name="plan_mixed_percentile_image", kind="plan", M=8192, width=1152, blocks=1, plan="mixed", R=256, p_ppm=999000, a_bits=8),
        # one denoising step of the whole 28-block stack under the seeded bit plan
        dict(name="stack_bit_plan_m16384", kind="plan", M=16384, width=1152, blocks=28, plan="bit_plan", R=1, p_ppm=0, a_bits=8),
        # a smaller batch of the same stack under a plan of the final kind: 4-bit groups of 32 to 288, 8-bit and FP16 layers
        dict(name="stack_final_plan_m4096", kind="plan", M=4096, width=1152, blocks=28, plan="final_plan", R=1, p_ppm=0, a_bits=8),
        # a block with everything between its linears that the library folds in
        dict(name="block_glue_m4096", kind="block", M=4096, width=1152, tokens=256, mlp_bits=8),
        # 6-bit codes with group scales and eq. (4)'s channel groups: 16 images, one scale per image and group of 128 inputs
        dict(name="grouped_w6_channel_scales", kind="grouped", M=4096, K=1152, N=3456, bits=6, group=128, R=256, channel=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _group_of(rng, K):
    fits = [g for g in W4_GROUPS if K % g == 0]
    return rng.choice(fits)


def _rows(rng, lo, hi):
    """Row count and rows per image: whole images half of the time, any count otherwise."""
    M = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        tokens = rng.choice([t for t in (64, 256, 1024) if t <= max(M, 64)])
        return max(1, M // tokens) * tokens, tokens
    return M, M


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "plan", "plan", "block", "grouped"))
    width = rng.choice(WIDTHS)
    if kind == "layer":
        bits = rng.choice((8, 8, 4, 4, 16))
        M, tokens = _rows(rng, 1, 16384)
        K, N = rng.choice(((width, width), (width, 3 * width), (width, 4 * width), (4 * width, width)))
        shape = rng.random()
        if shape < 0.15:
            # inputs that no K step divides (4-bit weights need whole groups); the cost of such a layer is bounded
            M, K, N = min(M, 2048), 8 * rng.randint(8, 200), _log_int(rng, 32, 1200)
            K = K if bits != 4 else 32 * max(2, K // 32)
            tokens = M
        elif shape < 0.4:
            N = _log_int(rng, 32, 4608)
        glue = rng.random()
        return dict(kind="layer", M=M, K=K, N=N, bits=bits, group=_group_of(rng, K) if bits == 4 else 0,
                    R=1 if bits == 16 else rng.choice((1, 1, 1, tokens)), act=1 if glue < 0.2 else 0, gated=0.2 <= glue < 0.4)
    if kind == "plan":
        M, tokens = _rows(rng, 128, 16384)
        percentile = rng.random() < 0.3
        return dict(kind="plan", M=M, width=width, blocks=rng.choice((1, 1, 2, 4)), plan=rng.choice(("w8", "mixed", "bit_plan", "final_plan")),
                    R=rng.choice((1, 1, tokens)), p_ppm=rng.choice((990000, 999000, 999900)) if percentile else 0,
                    a_bits=rng.choice((8, 6)) if percentile else 8)
    if kind == "block":
        tokens = rng.choice((64, 256, 1024))
        return dict(kind="block", M=tokens * _log_int(rng, 1, 16384 // tokens), width=width, tokens=tokens, mlp_bits=rng.choice((8, 4)))
    tokens = rng.choice((64, 256, 1024))
    K, N = rng.choice(((width, width), (width, 3 * width), (width, 4 * width), (4 * width, width)))
    group = _group_of(rng, K)
    # short images and very many groups are met at small batches only
    most = 16384 if tokens >= 256 and K // group <= 40 else 1024
    return dict(kind="grouped", M=tokens * _log_int(rng, 1, most // tokens), K=K, N=N, bits=rng.choice((3, 6)), group=group, R=tokens,
                channel=rng.random() < 0.7)


# ---------------------------------------------------------------- inputs

class _Maker:
    """Tensors of the distributions workload.py describes, drawn on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, std=1.0):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=self.g)

    def activations(self, M, K, sigma=1.0):
        """N(0, sigma^2), eight channels twenty times as large."""
        x = self.normal((M, K), sigma)
        x[:, torch.randint(0, K, (8,), generator=self.g, device="cuda")] *= 20.0
        return x.half()

    def hidden(self, M, K):
        """What the MLP's output layer sees: the GELU of a wide layer's outputs."""
        return torch.nn.functional.gelu(self.normal((M, K), 3.0), approximate="tanh").half()

    def ints(self, lo, hi, shape, dtype=torch.int8):
        return torch.randint(lo, hi + 1, shape, generator=self.g, device="cuda", dtype=dtype)

    def uniform(self, lo, hi, shape):
        return torch.empty(shape, device="cuda").uniform_(lo, hi, generator=self.g)

    def weights(self, K, N, bits, group):
        """Codes, scales and bias of one layer, as ql.Plan takes them."""
        bias = self.normal((N,), 0.02).half()
        if bits == 16:
            return dict(K=K, N=N, bits=16, w=self.normal((N, K), 0.02).half(), w_scale=None, bias=bias)
        if bits == 8:
            return dict(K=K, N=N, bits=8, w=self.ints(-127, 127, (N, K)), w_scale=self.uniform(1e-3, 1e-2, (N,)), bias=bias)
        # two nibbles per byte; every byte is a pair of codes in [-8, 7]
        return dict(K=K, N=N, bits=4, group=group, w=self.ints(0, 255, (N, K // 2), torch.uint8),
                    w_scale=self.uniform(1e-2, 1e-1, (N, K // group)).half(), bias=bias)


def _plan_layers(case):
    """[(K, N, bits, group)] of every layer of the case's blocks."""
    w, n = case["width"], case["blocks"]
    sizes = [(w, 3 * w), (w, w), (w, 4 * w), (4 * w, w)]
    if case["plan"] == "w8":
        marks = [(8, 0)] * (4 * n)
    elif case["plan"] == "mixed":
        marks = [(8, 0), (8, 0), (4, 128), (4, 128)] * n
    elif case["plan"] == "bit_plan":
        marks = [(p["bits"], p["group"]) for p in workload.bit_plan(n, protect=3 if n > 8 else 0)]
    else:
        marks = [(p["bits"], p["group"]) for p in workload.final_plan(n)]
    out = []
    for i, (bits, group) in enumerate(marks):
        K, N = sizes[i % 4]
        out.append((K, N, bits, 0 if bits != 4 else group if K % group == 0 else 128))
    return out


def prepare(case, seed):
    mk = _Maker(seed)
    kind, M = case["kind"], case["M"]
    s = dict(case=case)
    if kind == "layer":
        K, N, R = case["K"], case["N"], case["R"]
        s.update(x=mk.activations(M, K), layer=mk.weights(K, N, case["bits"], case["group"]),
                 y=torch.empty((M, N), dtype=torch.float16, device="cuda"))
        if case["bits"] != 16:
            s["ws"] = ql.workspace(ql.qlinear_workspace_bytes(M, K, R))
        if case["gated"]:
            s.update(residual=mk.normal((M, N)).half(), gate=mk.normal((1, N)).half())
    elif kind == "plan":
        shapes = _plan_layers(case)
        layers = [mk.weights(*l) for l in shapes]
        w, n = case["width"], case["blocks"]
        x = [mk.activations(M, w), mk.activations(M, w), mk.activations(M, w), mk.hidden(M, 4 * w)]
        y = [torch.empty((n, M, N), dtype=torch.float16, device="cuda") for (_, N, _, _) in shapes[:4]]
        plan = ql.Plan(layers, M_max=M)
        s.update(plan=plan, x_in=[x[i % 4] for i in range(4 * n)], y_out=[y[i % 4][i // 4] for i in range(4 * n)], y=y,
                 ws=ql.workspace(plan.workspace_bytes(M, case["R"])))
    elif kind == "block":
        w, t = case["width"], case["tokens"]
        sizes = [(w, 3 * w, 8), (w, w, 8), (w, 4 * w, case["mlp_bits"]), (4 * w, w, case["mlp_bits"])]
        s.update(x=mk.activations(M, w), attn=mk.activations(M, w), layers=[mk.weights(K, N, b, 128) for K, N, b in sizes],
                 mod=[mk.normal((M // t, w), 0.3).half() for _ in range(6)],
                 y=[torch.empty((M, N), dtype=torch.float16, device="cuda") for _, N, _ in sizes],
                 ws=ql.workspace(ql.qlinear_workspace_bytes(M, 4 * w, 1)))
    else:
        K, N, g, b = case["K"], case["N"], case["group"], case["bits"]
        s.update(x=mk.activations(M, K), w=mk.ints(-(1 << (b - 1)), (1 << (b - 1)) - 1, (N, K)),
                 w_scale=mk.uniform(1e-2, 1e-1, (N, K // g)).half(), bias=mk.normal((N,), 0.02).half(),
                 y=torch.empty((M, N), dtype=torch.float16, device="cuda"))
    return s


# ---------------------------------------------------------------- one pass

def _run_layer(s, case):
    l, R = s["layer"], case["R"]
    if case["bits"] == 16:
        return ql.qlinear_f16(s["x"], l["w"], l["bias"], act=case["act"], residual=s.get("residual"), gate=s.get("gate"),
                              gate_rows=case["M"], y=s["y"])
    if case["act"] or case["gated"]:
        return ql.qlinear_fused(s["x"], R, l["w"], l["w_scale"], l["bias"], bits=case["bits"], group=case["group"] or 128, act=case["act"],
                                residual=s.get("residual"), gate=s.get("gate"), gate_rows=case["M"], y=s["y"], ws=s["ws"])
    if case["bits"] == 8:
        return ql.qlinear_w8a8(s["x"], R, l["w"], l["w_scale"], l["bias"], y=s["y"], ws=s["ws"])
    return ql.qlinear_w4a8(s["x"], R, l["w"], l["w_scale"], l["bias"], y=s["y"], ws=s["ws"], group=case["group"])


def _run_block(s, case):
    t, ws = case["tokens"], s["ws"]
    qkv, proj, fc1, fc2 = s["layers"]
    y_qkv, y_proj, y_fc1, y_fc2 = s["y"]
    shift1, scale1, gate1, shift2, scale2, gate2 = s["mod"]
    n1 = ql.daq_quantize_ln(s["x"], 1, shift1, scale1, t)
    ql.qgemm_w8a8(n1["q"], n1["scales"], 1, qkv["w"], qkv["w_scale"], qkv["bias"], y=y_qkv)
    ql.qlinear_fused(s["attn"], 1, proj["w"], proj["w_scale"], proj["bias"], residual=s["x"], gate=gate1, gate_rows=t, y=y_proj, ws=ws)
    n2 = ql.daq_quantize_ln(y_proj, 1, shift2, scale2, t, want_h=True, want_q=False)
    bits = case["mlp_bits"]
    ql.qlinear_fused(n2["h"], 1, fc1["w"], fc1["w_scale"], fc1["bias"], bits=bits, act=ql.ACT_GELU_TANH, y=y_fc1, ws=ws)
    ql.qlinear_fused(y_fc1, 1, fc2["w"], fc2["w_scale"], fc2["bias"], bits=bits, residual=y_proj, gate=gate2, gate_rows=t, y=y_fc2, ws=ws)
    return list(s["y"])


def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        return _run_layer(state, case)
    if case["kind"] == "plan":
        if case["p_ppm"]:
            state["plan"].run_ex(state["x_in"], state["y_out"], case["M"], case["R"], state["ws"], p_ppm=case["p_ppm"], a_bits=case["a_bits"])
        else:
            state["plan"].run(state["x_in"], state["y_out"], case["M"], case["R"], state["ws"])
        return state["y"]
    if case["kind"] == "block":
        return _run_block(state, case)
    return ql.qlinear_grouped(state["x"], case["R"], state["w"], state["w_scale"], case["group"], state["bias"],
                              act_group=case["group"] if case["channel"] else 0, storage=8, y=state["y"])


# ---------------------------------------------------------------- work and tolerance

def _layer_work(M, K, N, bits, group):
    w = N * K * bits // 8 + (4 * N if bits == 8 else 2 * N * (K // group) if bits == 4 else 0) + 2 * N
    return dict(bytes=2 * M * K + w + 2 * M * N, flops=2 * M * N * K)


def work(case):
    kind, M = case["kind"], case["M"]
    if kind == "layer":
        r = _layer_work(M, case["K"], case["N"], case["bits"], case["group"])
        if case["gated"]:
            r["bytes"] += 2 * M * case["N"] + 2 * case["N"]
        return r
    if kind == "grouped":
        r = _layer_work(M, case["K"], case["N"], 8, 0)
        r["bytes"] += case["N"] * (2 * (case["K"] // case["group"]) - 4)
        return r
    if kind == "plan":
        parts = [_layer_work(M, *l) for l in _plan_layers(case)]
        # the three narrow inputs and the wide one are shared by all blocks
        shared = 2 * M * case["width"] * 7 * (case["blocks"] - 1)
        return dict(bytes=sum(p["bytes"] for p in parts) - shared, flops=sum(p["flops"] for p in parts))
    w, b = case["width"], case["mlp_bits"]
    parts = [_layer_work(M, w, 3 * w, 8, 0), _layer_work(M, w, w, 8, 0), _layer_work(M, w, 4 * w, b, 128), _layer_work(M, 4 * w, w, b, 128)]
    # outputs that the next stage reads again are not inputs of the block: y_proj feeds fc1, fc1 feeds fc2
    bytes_ = sum(p["bytes"] for p in parts) - 2 * M * w - 2 * M * 4 * w + 12 * (M // case["tokens"]) * w
    return dict(bytes=bytes_, flops=sum(p["flops"] for p in parts))


def tolerance(case):
    # fp16 outputs of one rounding (2^-11); in a block the LayerNorm's fp32 sums may move an fp16 value by a step and an
    # 8-bit code by one, and the next layers see it
    return {"rel": 3e-3} if case["kind"] == "block" else {"rel": 1e-3}
