"""The work that a user of the HALO linear layer has it do, as cases that can be timed and compared.

Kinds of work:
  forward  halo_linear_fwd on X and W as they come (an evaluation pass during training)
  infer    halo_linear_fwd on a weight that was rotated and quantised once: decode (a few tokens) and prefill
  step     halo_linear_fwd + halo_linear_bwd of one linear, what every training step runs
  layer    the step of the seven linears of one decoder layer; q/k/v and gate/up share one quantised activation
  peft     halo_peft_fwd + halo_peft_bwd: frozen quantised weight, LoRA adapters
  mx6      the MXFP6 forward product: both operands quantised, then multiplied

As in a training loop, the workspace is kept from pass to pass, and outputs and saved codes are new in every pass.
"""
import math

import torch

from paper_2501_02625_amd import binding, inputs

DEVICE = "cuda:0"
OUTLIERS = 0.001          # share of the activation's channels that are outliers
LAYER = inputs.CONFIGS["c4"].linears


def listed():
    return [
        # The smallest forward call: 128 tokens, 512 channels, the shape of the paper's outlier figure (config c1).
        _case("forward", 128, 512, 512, name="forward_128x512x512"),
        # Decode with a resident INT8 weight: one tile of 16 tokens through a 4096 x 4096 projection.
        _case("infer", 16, 4096, 4096, name="decode_16x4096x4096"),
        # Prefill with a resident INT8 weight: batch 4 x 512 tokens through an up-projection.
        _case("infer", 2048, 4096, 14336, name="prefill_2048x4096x14336"),
        # A small training step with left- and right-hand rotations and fp32 outputs, the size of the smoke test.
        _case("step", 256, 1024, 512, level=2, out="fp32", name="step_l2_256x1024x512"),
        # Sizes that no tile divides: tokens and channels odd multiples of 16, Hadamard blocks of 512.
        _case("step", 1040, 5632, 2320, out="fp32", name="step_ragged_1040x5632x2320"),
        # Attention projection, batch 4 x 512 tokens, HALO-1 (config c2, the benchmark's workload).
        _case("step", 2048, 4096, 4096, name="step_l1_2048x4096x4096"),
        # The same with the paper's own quantiser, one scale per tensor (config c7).
        _case("step", 2048, 4096, 4096, scale="tensor", name="step_tensor_2048x4096x4096"),
        # Down-projection, block-diagonal rotation 7 x 2048 over K = 14336, HALO-2 (config c3).
        _case("step", 4096, 14336, 4096, level=2, name="step_l2_4096x14336x4096"),
        # The same with one Kronecker block H_512 (x) H_28 over K = 14336 (config c6).
        _case("step", 4096, 14336, 4096, level=2, block=14336, name="step_kron_4096x14336x4096"),
        # LoRA fine-tuning step, rank 16, HALO-2 (config c8).
        _case("peft", 4096, 4096, 4096, level=2, rank=16, name="peft_r16_4096x4096x4096"),
        # MXFP6 forward product (config c5).
        _case("mx6", 8192, 4096, 4096, name="mx6_8192x4096x4096"),
        # All seven linears of a decoder layer, 8192 tokens, HALO-2, forward and backward (config c4).
        _case("layer", 8192, 4096, 14336, level=2, name="layer_l2_8192"),
    ]


def _case(kind, b, m, n, level=1, scale="row", block=0, out="bf16", rank=0, name=None):
    """b tokens, m in-features, n out-features.  block: right-hand Hadamard block, 0 = the layer's default."""
    c = dict(kind=kind, b=b, m=m, n=n, level=level, scale=scale, block=block, out=out, rank=rank)
    if name:
        c["name"] = name
    return c


def _log(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _width(rng, step, lo=256):
    """A layer width: half of the time one of the usual ones, otherwise any multiple of `step`."""
    if rng.random() < 0.5:
        return rng.choice([512, 1024, 1536, 2048, 3072, 4096, 5120, 8192, 14336])
    return _log(rng, lo, 14336, step)


def draw(rng):
    kind = rng.choices(["forward", "infer", "step", "peft", "mx6"], [2, 4, 8, 2, 2])[0]
    # tokens: whole sequences half of the time (multiples of 256), otherwise any multiple of 16
    b = _log(rng, 256, 8192, 256) if rng.random() < 0.5 else _log(rng, 16 if kind in ("infer", "mx6") else 128, 8192, 16)
    if kind == "mx6":
        return _case("mx6", b, _width(rng, 128), _width(rng, 16))
    if kind == "peft":
        return _case("peft", b, _width(rng, 64), _width(rng, 64), level=rng.choice([1, 2, 2]), rank=rng.choice([8, 16, 32, 64]))
    m, n = _width(rng, 64), _width(rng, 16)
    out = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    if kind in ("forward", "infer"):
        return _case(kind, b, m, n, out=out)
    scale = rng.choice(["row", "row", "row", "tensor"])
    block = 0
    if rng.random() < 0.12:
        m = rng.choice([1792, 3584, 7168, 14336])
        block = m
    return _case("step", b, m, n, level=rng.choice([0, 1, 1, 2, 2, 2]) if not block else rng.choice([1, 2]), scale=scale,
                 block=block, out=out)


# ---------------------------------------------------------------------------------------------- inputs
def _activations(g, b, m):
    """N(0, 1) with a few outlier channels, x50."""
    x = torch.randn((b, m), generator=g, device=DEVICE)
    count = max(1, round(OUTLIERS * m))
    idx = torch.randperm(m, generator=g, device=DEVICE)[:count]
    x[:, idx] *= inputs.OUTLIER_GAIN
    return x.to(torch.bfloat16)


def _weights(g, n, m):
    return (torch.randn((n, m), generator=g, device=DEVICE) * inputs.WEIGHT_STD).to(torch.bfloat16)


def _errors(g, b, n):
    """Heavy-tailed output gradients: 1e-3 x Student-t with three degrees of freedom."""
    s = torch.zeros((b, n), device=DEVICE)
    for _ in range(inputs.ERROR_DOF):
        s += torch.randn((b, n), generator=g, device=DEVICE).square_()
    z = torch.randn((b, n), generator=g, device=DEVICE)
    return (z / (s / inputs.ERROR_DOF).sqrt_() * inputs.ERROR_SCALE).to(torch.bfloat16)


def _desc(case, m=None, n=None):
    return binding.make_desc(case["b"], m or case["m"], n or case["n"], case["level"],
                             torch.float32 if case["out"] == "fp32" else torch.bfloat16, had_block_m=case["block"],
                             scale_mode=binding.HALO_SCALE_PER_TENSOR if case["scale"] == "tensor"
                             else binding.HALO_SCALE_PER_ROW)


def _right_block(case):
    m = case["m"]
    return 0 if case["level"] == 0 else case["block"] or min(m & -m, 4096)


def _bytes(n):
    return torch.empty((max(int(n), 16),), dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    kind, b, m, n = case["kind"], case["b"], case["m"], case["n"]
    s = {"kind": kind}
    if kind == "layer":
        s["linears"], size, acts = [], 0, {}
        for lin in LAYER:
            owner = lin.shares_input_with or lin.name
            if owner == lin.name:
                acts[owner] = _activations(g, b, lin.m)
            desc = _desc(case, lin.m, lin.n)
            size = max(size, binding.halo_linear_workspace_bytes(desc))
            s["linears"].append((lin, desc, acts[owner] if owner == lin.name else None, _weights(g, lin.n, lin.m),
                                 _errors(g, b, lin.n)))
        s["workspace"] = _bytes(size)
        return s
    s["X"] = _activations(g, b, m)
    W = _weights(g, n, m)
    if kind == "mx6":
        s["W"], s["block"] = W, _right_block(case)
        return s
    s["desc"] = _desc(case)
    if kind == "peft":
        r = case["rank"]
        s["Wq"], s["s_w"] = binding.halo_hadamard_quant(W, had_block=_right_block(case))
        s["U"] = ((torch.rand((r, m), generator=g, device=DEVICE) * 2 - 1) / math.sqrt(m)).to(torch.bfloat16)
        s["V"] = (torch.randn((n, r), generator=g, device=DEVICE) * inputs.ADAPTER_V_STD).to(torch.bfloat16)
        s["E"] = _errors(g, b, n)
        s["workspace"] = _bytes(binding.halo_peft_workspace_bytes(s["desc"], r))
        return s
    if kind == "infer":
        Wq, s_w = binding.halo_hadamard_quant(W, had_block=_right_block(case))
        s["state"] = binding.LinearState(torch.empty((b, m), dtype=torch.int8, device=DEVICE),
                                         torch.empty((b,), dtype=torch.float32, device=DEVICE), Wq, s_w)
        return s
    s["W"] = W
    if kind == "step":
        s["E"] = _errors(g, b, n)
    s["workspace"] = _bytes(binding.halo_linear_workspace_bytes(s["desc"]))
    return s


# ---------------------------------------------------------------------------------------------- one pass
def _saved(st):
    return [st.Xq, st.s_x, st.Wq, st.s_w]


def run(s):
    kind = s["kind"]
    if kind == "infer":
        Y, st = binding.halo_linear_fwd(s["desc"], s["X"], None, state=s["state"])
        return [Y, st.Xq, st.s_x]
    if kind == "forward":
        Y, st = binding.halo_linear_fwd(s["desc"], s["X"], s["W"], workspace=s["workspace"])
        return [Y] + _saved(st)
    if kind == "step":
        Y, st = binding.halo_linear_fwd(s["desc"], s["X"], s["W"], workspace=s["workspace"])
        EX, G = binding.halo_linear_bwd(s["desc"], s["E"], st, workspace=s["workspace"])
        return [Y] + _saved(st) + [EX, G]
    if kind == "peft":
        Y, T = binding.halo_peft_fwd(s["desc"], s["X"], s["Wq"], s["s_w"], s["U"], s["V"], workspace=s["workspace"])
        EX, GU, GV = binding.halo_peft_bwd(s["desc"], s["E"], s["X"], T, s["Wq"], s["s_w"], s["U"], s["V"],
                                           workspace=s["workspace"])
        return [Y, T, EX, GU, GV]
    if kind == "mx6":
        xq, sx = binding.halo_mx6_quant(s["X"], had_block=s["block"])
        wq, sw = binding.halo_mx6_quant(s["W"], had_block=s["block"])
        return [binding.halo_gemm_mx6(xq, sx, wq, sw, out_dtype=torch.bfloat16), xq, sx, wq, sw]
    # layer: all forward passes, then all backward passes
    out, states = [], {}
    for lin, desc, X, W, E in s["linears"]:
        if X is None:
            src = states[lin.shares_input_with]
            st = binding.LinearState(src.Xq, src.s_x, torch.empty((lin.n, lin.m), dtype=torch.int8, device=W.device),
                                     torch.empty((lin.n,), dtype=torch.float32, device=W.device))
            Y, st = binding.halo_linear_fwd(desc, None, W, state=st, workspace=s["workspace"])
        else:
            Y, st = binding.halo_linear_fwd(desc, X, W, workspace=s["workspace"])
            out += [st.Xq, st.s_x]
        states[lin.name] = st
        out += [Y, st.Wq, st.s_w]
    for lin, desc, X, W, E in reversed(s["linears"]):
        EX, G = binding.halo_linear_bwd(desc, E, states[lin.name], workspace=s["workspace"])
        out += [EX, G]
    return out


# ---------------------------------------------------------------------------------------------- what it takes
def work(case):
    kind, b, m, n = case["kind"], case["b"], case["m"], case["n"]
    o = 4 if case["out"] == "fp32" else 2
    if kind == "layer":
        total = {"bytes": 0, "flops": 0}
        for lin in LAYER:
            w = work(dict(case, kind="step", m=lin.m, n=lin.n))
            total["flops"] += w["flops"]
            # an activation that another linear has quantised is neither read nor written again
            total["bytes"] += w["bytes"] - ((3 * b * lin.m + 4 * b) if lin.shares_input_with else 0)
        return total
    if kind == "mx6":
        codes = 25 / 32
        return {"bytes": (2 + codes) * (b * m + n * m) + 2 * b * n, "flops": 2 * b * n * m}
    if kind == "peft":
        r = case["rank"]
        thin = 2 * r * (m + n) + 4 * b * r + 4 * r * (m + n)
        return {"bytes": 2 * b * m + n * m + 4 * n + 2 * b * n + o * (b * n + b * m) + thin,
                "flops": 4 * b * n * m + 12 * b * r * (n + m)}
    quant_x, quant_w = 3 * b * m + 4 * b, 3 * n * m + 4 * n
    if kind == "infer":
        return {"bytes": quant_x + n * m + 4 * n + o * b * n, "flops": 2 * b * n * m}
    if kind == "forward":
        return {"bytes": quant_x + quant_w + o * b * n, "flops": 2 * b * n * m}
    return {"bytes": quant_x + quant_w + 2 * b * n + o * (b * n + b * m + n * m), "flops": 6 * b * n * m}


def tolerance(case):
    # bf16 outputs are rounded once at the end (half an ulp is 2^-9); the codes have to be the same bytes
    if case["out"] == "bf16":
        return {"rel": 4e-3, "max": 2e-2, "differ": 0.0}
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
