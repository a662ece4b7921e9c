"""The work this library is used for, as cases that can be timed and whose outputs can be compared.

Entry points: zs_gemm (FP32 output), zs_gemm_bf16, zs_linear (fused below its crossover, decompress
+ dense GEMM above), zs_decompress, zs_encode_device.  Shapes are the LLaMA-3.1 8B / 70B linear
layers of paper_2603_17435_amd/inputs.py and the 128256 x 4096 LM head of the benchmark; weight
laws are the seeded ones of the tests (Gaussian, Student-t, per-row scales, outliers), drawn on the GPU.
A case is {"op", "N", "K", "M", "law"}; "decode_step" is one decoder layer: QKV, O, GateUp, Down.
"""
import math

import torch

from paper_2603_17435_amd import binding, inputs

LAYERS_8B = {name: (n, k) for name, n, k in inputs.LLAMA3_8B_LAYERS}
LAYERS_70B = {name: (n, k) for name, n, k in inputs.LLAMA3_70B_LAYERS}
STEP_LAYERS = ("qkv", "o", "gate_up", "down")

# sizes a drawn case may take: no drawn case costs more than the largest listed one of its kind
MAX_GEMM_ELEMS = 128256 * 4096
MAX_LINEAR_MACS = 2048 * 28672 * 4096
MAX_CODEC_ELEMS = 28672 * 4096


def _case(name, op, shape, m, law="gauss"):
    return {"name": name, "op": op, "N": shape[0], "K": shape[1], "M": m, "law": law}


def listed():
    return [
        # the smallest call of a decode step: the K (or V) projection for a single sequence; latency
        _case("gemm_kv_m1", "gemm", (1024, 4096), 1),
        # a small attention projection for a few sequences, BF16 activations out as a model keeps them
        _case("bf16_qkv_m7", "gemm_bf16", LAYERS_8B["qkv"], 7),
        # one whole decoder layer's weights for 32 sequences: the benchmark's step
        {"name": "decode_step_m32", "op": "decode_step", "N": 0, "K": 0, "M": 32, "law": "gauss"},
        # the widest layer of a block for 16 sequences
        _case("gemm_gate_up_m16", "gemm", LAYERS_8B["gate_up"], 16),
        # a larger, ragged decode batch
        _case("bf16_gate_up_m50", "gemm_bf16", LAYERS_8B["gate_up"], 50),
        # a short prompt, or decode with speculative tokens: above the skinny kernels, below the crossover
        _case("linear_down_m200", "linear", LAYERS_8B["down"], 200),
        # a prefill chunk: decompression followed by the dense GEMM
        _case("linear_gate_up_m2048", "linear", LAYERS_8B["gate_up"], 2048),
        # logits of one sequence
        _case("bf16_lm_head_m1", "gemm_bf16", (128256, 4096), 1),
        # the larger model family, decode batch through the stage-aware entry point
        _case("linear_down70b_m32", "linear", LAYERS_70B["down"], 32),
        # weights whose rows differ in scale: a third of the elements take the fallback path
        _case("gemm_rowscale_down_m16", "gemm", LAYERS_8B["down"], 16, "rowscale"),
        # weights unpacked for another consumer
        _case("decompress_gate_up", "decompress", LAYERS_8B["gate_up"], 0),
        # weights packed on the GPU when a model is loaded
        _case("encode_gate_up", "encode", LAYERS_8B["gate_up"], 0),
    ]


def _log_size(rng, lo, hi, step):
    return step * max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step))


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm_bf16", "gemm_bf16", "linear", "linear", "decode_step", "decompress", "encode"])
    law = rng.choice(["gauss", "gauss", "gauss", "student_t", "rowscale", "outliers"])
    if op == "decode_step":
        return {"op": op, "N": 0, "K": 0, "M": rng.randint(1, 32), "law": law}
    limit = MAX_CODEC_ELEMS if op in ("decompress", "encode", "linear") else MAX_GEMM_ELEMS
    while True:
        n, k = _log_size(rng, 1024, 57344, 64), _log_size(rng, 1024, 28672, 64)
        if n * k <= limit:
            break
    m = 0
    if op in ("gemm", "gemm_bf16"):
        m = _log_size(rng, 1, 64, 1)
    elif op == "linear":
        m = min(_log_size(rng, 1, 4096, 1), MAX_LINEAR_MACS // (n * k))
    return {"op": op, "N": n, "K": k, "M": m, "law": law}


def _weights(n, k, law, gen):
    """[n, k] BF16 weights of the law; the scale of all of them is 0.02."""
    w = torch.randn(n, k, generator=gen, device="cuda", dtype=torch.float32)
    if law == "student_t":  # three degrees of freedom
        chi2 = torch.zeros_like(w)
        for _ in range(3):
            chi2 += torch.randn(n, k, generator=gen, device="cuda", dtype=torch.float32).square_()
        w *= chi2.div_(3.0).rsqrt_()
    elif law == "outliers":  # one weight in a thousand is fifty times larger
        w.mul_(torch.where(torch.rand(n, k, generator=gen, device="cuda") < 1e-3, 50.0, 1.0))
    elif law == "rowscale":  # row scales log-uniform over three decades
        w *= torch.exp(torch.rand(n, 1, generator=gen, device="cuda") * math.log(1e3) - math.log(1e3))
    return w.mul_(0.02).to(torch.bfloat16)


def _packed(n, k, law, gen):
    """The matrix as a program that serves it holds it: blob on the GPU, descriptor on the host."""
    w = _weights(n, k, law, gen)
    cap = binding.zs_encode_bound(n, k)
    blob = torch.empty(cap, dtype=torch.uint8, device="cuda")
    scratch = torch.empty(binding.ZS_ENCODE_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")
    desc = binding.zs_encode_device(w, n, k, blob, cap, scratch)
    return blob[:desc.total_bytes].clone(), desc


def _gemm_state(n, k, m, law, gen, op):
    blob, desc = _packed(n, k, law, gen)
    size = binding.zs_linear_workspace(desc, m) if op == "linear" else binding.zs_gemm_workspace(desc, min(m, 64))
    decoupled = op == "linear" and binding.zs_linear_path(desc, m) == binding.ZS_PATH_DECOUPLED
    return {
        "blob": blob, "desc": desc, "M": m,
        "A": torch.randn(m, k, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16),
        "C": torch.empty(m, n, dtype=torch.bfloat16 if op == "gemm_bf16" else torch.float32, device="cuda"),
        # the fused kernels' scratch starts from zero once; the decompressed weights need not
        "ws": (torch.empty if decoupled else torch.zeros)(max(size, 256), dtype=torch.uint8, device="cuda"),
    }


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    op, n, k, m, law = case["op"], case["N"], case["K"], case["M"], case["law"]
    if op == "encode":
        cap = binding.zs_encode_bound(n, k)
        # zeroed: the packer leaves what lies beyond the blob as it was, and the whole buffer is returned
        return {"op": op, "W": _weights(n, k, law, gen), "N": n, "K": k, "cap": cap,
                "blob": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                "ws": torch.empty(binding.ZS_ENCODE_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")}
    if op == "decompress":
        blob, desc = _packed(n, k, law, gen)
        return {"op": op, "blob": blob, "desc": desc, "out": torch.empty(n, k, dtype=torch.int16, device="cuda")}
    if op == "decode_step":
        layers = [_gemm_state(*LAYERS_8B[name], m, law, gen, "gemm") for name in STEP_LAYERS]
        ws = max((s["ws"] for s in layers), key=lambda t: t.numel())  # one scratch serves every layer
        for s in layers:
            s["ws"] = ws
        return {"op": op, "layers": layers}
    return {"op": op, **_gemm_state(n, k, m, law, gen, op)}


def _gemm(s):
    binding.zs_gemm(s["desc"], s["blob"], s["A"], s["C"], s["M"], workspace_dev=s["ws"], workspace_bytes=s["ws"].numel())
    return s["C"]


def run(state):
    op = state["op"]
    if op == "gemm":
        return _gemm(state)
    if op == "decode_step":
        return [_gemm(s) for s in state["layers"]]
    if op == "gemm_bf16":
        binding.zs_gemm_bf16(state["desc"], state["blob"], state["A"], state["C"], state["M"], workspace_dev=state["ws"],
                             workspace_bytes=state["ws"].numel())
        return state["C"]
    if op == "linear":
        binding.zs_linear(state["desc"], state["blob"], state["A"], state["C"], state["M"], workspace_dev=state["ws"],
                          workspace_bytes=state["ws"].numel())
        return state["C"]
    if op == "decompress":
        binding.zs_decompress(state["desc"], state["blob"], state["out"])
        return state["out"]
    d = binding.zs_encode_device(state["W"], state["N"], state["K"], state["blob"], state["cap"], state["ws"])
    return {"blob": state["blob"], "total_bytes": d.total_bytes, "base_exp": d.base_exp, "n_high": d.n_high,
            "n_fallback": d.n_fallback, "h_bytes": d.h_bytes, "l_bytes": d.l_bytes, "max_h_units": d.max_h_units, "max_l_units": d.max_l_units}


# bytes per weight of the packed matrix, (19 - 8 r) bits with r the share of weights inside the
# seven-exponent window of each law (measured on these shapes), without offsets and padding
_R = {"gauss": 0.979, "student_t": 0.956, "rowscale": 0.672, "outliers": 0.978}


def work(case):
    op, m = case["op"], case["M"]
    shapes = [LAYERS_8B[name] for name in STEP_LAYERS] if op == "decode_step" else [(case["N"], case["K"])]
    packed = (19.0 - 8.0 * _R[case["law"]]) / 8.0
    total, flops = 0.0, 0.0
    for n, k in shapes:
        total += packed * n * k
        if op in ("decompress", "encode"):
            total += 2.0 * n * k
        else:
            total += 2.0 * m * k + (2.0 if op == "gemm_bf16" else 4.0) * m * n
            flops += 2.0 * m * n * k
    return {"bytes": total, "flops": flops}


def exact(case, seed):
    """The products in float64 on the weights and activations that `prepare` draws from this seed."""
    if case["op"] in ("decompress", "encode"):
        return None  # bytes
    gen = torch.Generator(device="cuda").manual_seed(seed)
    step = case["op"] == "decode_step"
    out = []
    for n, k in [LAYERS_8B[name] for name in STEP_LAYERS] if step else [(case["N"], case["K"])]:
        w = _weights(n, k, case["law"], gen)
        a = torch.randn(case["M"], k, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
        out.append(a.double() @ w.double().t())
    return out if step else out[0]


def tolerance(case):
    """Measured against the products in float64 over the listed cases and drawn ones: FP32 results
    differ by at most 6.5e-7 (largest element 1e-5 of the RMS), BF16 results from the rounded
    float64 ones, and from themselves in another order of summation, by 3e-5 (a value next to a
    rounding boundary moves by one step, at most 2^-7 of itself); about four times that is allowed."""
    if case["op"] in ("decompress", "encode"):
        return "exact"
    if case["op"] == "gemm_bf16":
        return {"rel": 1.5e-4, "max": 2e-2}
    return {"rel": 2.5e-6, "max": 4e-5}
