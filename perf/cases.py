"""The work a user of this library has it do, as cases that can be timed and checked.

Every case is a dict of plain values; `kind` names the part of the public interface it goes through:

  linear    one product C = epilogue(A . B) by gemm_create / gemm_run: a layer's forward pass, a decode step, a batch of
            small products.  B is stored N x K (`b` = "col", a layer's weight) or K x N (`b` = "row", a plain matrix product).
  backward  the two products of a linear layer's backward pass over `M` tokens, weight N x K: the input's gradient
            dY . W (M x K) and the weight's gradient dY^T . X (N x K).
  splitk    one product by gemm_create_splitk / gemm_run_workspace, with the library's own number of slices.
  rope      the rotary embedding of a layer's query and key tensors by rope_apply, tensors as the projection leaves them.

A plan, the weights, the outputs' buffers and a workspace are what a program keeps from step to step: `prepare` makes them.
"""
import math

import torch

import paper_2603_12440_amd as g

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn}
CODE = {"f32": g.F32, "bf16": g.BF16, "f16": g.F16, "f8": g.F8E4M3}
SIZE = {"f32": 4, "bf16": 2, "f16": 2, "f8": 1}


def _linear(name, M, N, K, dtype="bf16", out="bf16", b="col", epilogue="none", batch=1):
    return {"name": name, "kind": "linear", "M": M, "N": N, "K": K, "dtype": dtype, "out": out, "b": b,
            "epilogue": epilogue, "batch": batch}


def listed():
    return [
        # the smallest call: one small fp32 product, where the launch and the latency of a single pass over K count
        _linear("f32_256", 256, 256, 256, dtype="f32", out="f32", b="row"),
        # an ordinary fp32 product with both operands row-major, sizes that fill no tile evenly
        _linear("f32_2000x1500x1100", 2000, 1500, 1100, dtype="f32", out="f32", b="row"),
        # decode, one sequence: a matrix-vector product with a layer's weight
        _linear("decode_m1_8192x8192", 1, 8192, 8192),
        # decode, sixteen sequences, the widest weight
        _linear("decode_m16_28672x8192", 16, 28672, 8192),
        # decode, 64 sequences: the query/key/value projection of an LLM layer
        _linear("decode_m64_6144x4096", 64, 6144, 4096),
        # prefill of one prompt of 777 tokens: the feed-forward layer with its bias and GELU
        _linear("ffn_gelu_777x14336x4096", 777, 14336, 4096, epilogue="bias_gelu_erf"),
        # the largest product of the benchmark
        _linear("square_8192", 8192, 8192, 8192),
        # training: backward pass of a projection over a packed batch of 3001 tokens
        {"name": "backward_3001x6144x4096", "kind": "backward", "M": 3001, "N": 6144, "K": 4096, "dtype": "bf16"},
        # many small products at once
        _linear("batched_64x512x512x128", 512, 512, 128, batch=64),
        # 8-bit operands: the feed-forward layer over 4096 tokens
        _linear("f8_llm_4096x14336x4096", 4096, 14336, 4096, dtype="f8"),
        # few outputs, a very long K
        {"name": "splitk_512x512x32768", "kind": "splitk", "M": 512, "N": 512, "K": 32768, "dtype": "bf16", "out": "bf16"},
        # rotary embedding of a 1B-parameter decoder layer's queries and keys, long sequences
        {"name": "rope_b8_s4096_d64", "kind": "rope", "batch": 8, "heads_q": 32, "heads_k": 8, "seq": 4096, "head_dim": 64,
         "dtype": "bf16"},
    ]


def _spread(rng, lo, hi, step=1):
    """A size from lo to hi, even over its logarithm, a multiple of step."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return min(hi // step * step, max(-(-lo // step) * step, int(n) // step * step))


def draw(rng):
    kind = rng.choice(["linear", "linear", "decode", "batch", "backward", "backward", "f8", "f32", "splitk", "rope"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16"])
    out = rng.choice([dtype, dtype, dtype, "f32"])
    epilogue = rng.choice(["none", "none", "bias", "bias_gelu_erf", "bias_gelu_tanh", "bias_relu"])
    while True:
        if kind == "linear":            # forward of a layer: few rows to the largest; a few with odd K or a K x N weight
            c = _linear("", _spread(rng, 17, 8192), _spread(rng, 256, 16384), _spread(rng, 256, 16384, 8), dtype, out,
                        rng.choice(["col", "col", "col", "row"]), epilogue)
            if rng.random() < 0.15:
                c["K"] += rng.randrange(1, 8)
        elif kind == "decode":
            c = _linear("", rng.randrange(1, 17), _spread(rng, 1024, 28672), _spread(rng, 1024, 8192, 8), dtype, out,
                        "col", epilogue)
        elif kind == "batch":
            c = _linear("", _spread(rng, 64, 1024), _spread(rng, 64, 1024), _spread(rng, 32, 512, 8), dtype, dtype, "col",
                        "none", _spread(rng, 2, 256))
        elif kind == "backward":
            c = {"kind": "backward", "M": _spread(rng, 64, 8192), "N": _spread(rng, 256, 8192, 8),
                 "K": _spread(rng, 256, 8192, 8), "dtype": dtype}
        elif kind == "f8":
            c = _linear("", _spread(rng, 16, 8192), _spread(rng, 256, 16384), _spread(rng, 256, 16384, 16), "f8",
                        rng.choice(["bf16", "bf16", "f32"]), "col", epilogue)
        elif kind == "f32":
            c = _linear("", _spread(rng, 16, 3000), _spread(rng, 16, 3000), _spread(rng, 16, 3000), "f32", "f32",
                        rng.choice(["row", "col"]), epilogue)
        elif kind == "splitk":
            c = {"kind": "splitk", "M": _spread(rng, 64, 1024, 8), "N": _spread(rng, 64, 1024, 8),
                 "K": _spread(rng, 4096, 65536, 512), "dtype": dtype, "out": out}
        else:
            heads = rng.choice([8, 16, 32])
            c = {"kind": "rope", "batch": rng.randrange(1, 9), "heads_q": heads, "heads_k": rng.choice([2, 4, 8]),
                 "seq": _spread(rng, 128, 8192), "head_dim": rng.choice([64, 128]), "dtype": dtype}
        c.pop("name", None)
        w = work(c)
        if w["flops"] < (4e11 if c["kind"] == "backward" or c.get("b") == "row" or c.get("K", 0) % 8 else 1.1e12) and w["bytes"] < 5e8:
            return c


def work(case):
    c = case
    if c["kind"] == "rope":
        n = c["batch"] * (c["heads_q"] + c["heads_k"]) * c["seq"] * c["head_dim"]
        return {"bytes": 2 * SIZE[c["dtype"]] * n + 2 * 4 * c["seq"] * c["head_dim"], "flops": 3 * n}
    M, N, K, e, batch = c["M"], c["N"], c["K"], SIZE[c["dtype"]], c.get("batch", 1)
    if c["kind"] == "backward":         # dY, W and X read once; dX and dW written
        return {"bytes": e * (M * N + N * K + M * K + M * K + N * K), "flops": 4 * M * N * K}
    bias = 4 * N if "bias" in c.get("epilogue", "") else 0
    return {"bytes": batch * (e * (M * K + K * N) + SIZE[c["out"]] * M * N) + bias, "flops": 2 * M * N * K * batch}


def tolerance(case):
    # Four times the 2-norm error measured against 64 bits over the drawn cases.  16-bit results: one rounding, 1.7e-3 (bf16)
    # and 2.1e-4 (fp16).  32-bit results: the sums' own rounding, up to 9.2e-7; with 8-bit operands, whose products the
    # matrix cores add with fewer bits, 1.1e-5.
    out = case["dtype"] if case["kind"] in ("rope", "backward") else case["out"]
    return {"rel": {"bf16": 7e-3, "f16": 9e-4, "f32": 4.5e-5 if case["dtype"] == "f8" else 4e-6}[out]}


def _inputs(case, seed):
    """The operands alone, from the seed."""
    c = case
    rng = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0, dtype=None):
        t = torch.randn(*shape, generator=rng, device="cuda", dtype=torch.float32)
        return t.mul_(scale).to(TORCH[dtype or c["dtype"]])

    if c["kind"] == "rope":
        B, S, D = c["batch"], c["seq"], c["head_dim"]
        first = int(torch.randint(0, 1000, (1,), generator=rng, device="cuda"))     # position of the first token
        pos = torch.arange(first, first + S, device="cuda", dtype=torch.float64)
        freq = 500000.0 ** (-2.0 * torch.arange(D // 2, device="cuda", dtype=torch.float64) / D)
        angle = torch.cat([pos[:, None] * freq, pos[:, None] * freq], dim=1)
        return {"q": normal(B, S, c["heads_q"], D), "k": normal(B, S, c["heads_k"], D),
                "cos": angle.cos().float(), "sin": angle.sin().float()}
    M, N, K = c["M"], c["N"], c["K"]
    if c["kind"] == "backward":         # activations of order 1, weights 0.02, gradients small
        return {"X": normal(M, K), "W": normal(N, K, scale=0.02), "dY": normal(M, N, scale=0.01)}
    batch = c.get("batch", 1)
    scale = {"f8": 0.25, "f32": 1.0}.get(c["dtype"], 0.02)
    d = {"A": normal(batch, M, K), "B": normal(batch, *((N, K) if c.get("b", "col") == "col" else (K, N)), scale=scale)}
    if "bias" in c.get("epilogue", ""):
        d["bias"] = normal(N, scale=0.1, dtype="f32")
    return d


def prepare(case, seed):
    c = case
    s = dict(_inputs(case, seed), kind=c["kind"])
    dt = TORCH[c["dtype"]]
    if c["kind"] == "rope":
        B, S, D = c["batch"], c["seq"], c["head_dim"]
        s["desc"] = g.RopeDesc(B, S, D, dtype=CODE[c["dtype"]], table_dtype=g.F32)
        s["qy"], s["ky"] = torch.empty_like(s["q"]), torch.empty_like(s["k"])
        s["tensors"] = []
        for x, y, h in ((s["q"], s["qy"], c["heads_q"]), (s["k"], s["ky"], c["heads_k"])):
            strides = (S * h * D, D, h * D)
            s["tensors"].append(g.RopeTensor(x, y, h, strides, strides))
        return s
    M, N, K = c["M"], c["N"], c["K"]
    if c["kind"] == "backward":
        s["dX"] = torch.empty(M, K, dtype=dt, device="cuda")
        s["dW"] = torch.empty(N, K, dtype=dt, device="cuda")
        # dX = dY . W: W is stored N x K, the product runs over N
        s["plan_x"] = g.gemm_create(g.GemmDesc(M, K, N, dtype=CODE[c["dtype"]], layout_b=g.ROW_MAJOR))
        # dW = dY^T . X: the product runs over the tokens
        s["plan_w"] = g.gemm_create(g.GemmDesc(N, K, M, dtype=CODE[c["dtype"]], layout_a=g.COL_MAJOR, layout_b=g.ROW_MAJOR))
        return s
    batch = c.get("batch", 1)
    desc = g.GemmDesc(M, N, K, dtype=CODE[c["dtype"]], dtype_c=CODE[c["out"]], batch=batch,
                      layout_b=g.COL_MAJOR if c.get("b", "col") == "col" else g.ROW_MAJOR,
                      epilogue=g.EPILOGUES[c.get("epilogue", "none")])
    s["C"] = torch.empty(batch, M, N, dtype=TORCH[c["out"]], device="cuda")
    s.setdefault("bias", None)
    if c["kind"] == "splitk":
        s["plan"] = g.gemm_create_splitk(desc)
        s["workspace"] = torch.empty(max(g.gemm_workspace_bytes(s["plan"]), 16), dtype=torch.uint8, device="cuda")
    else:
        s["plan"] = g.gemm_create(desc)
    return s


def run(state):
    s = state
    if s["kind"] == "rope":
        g.rope_apply(s["desc"], s["tensors"], s["cos"], s["sin"])
        return [s["qy"], s["ky"]]
    if s["kind"] == "backward":
        g.gemm_run(s["plan_x"], s["dY"], s["W"], s["dX"])
        g.gemm_run(s["plan_w"], s["dY"], s["X"], s["dW"])
        return [s["dX"], s["dW"]]
    if s["kind"] == "splitk":
        g.gemm_run_workspace(s["plan"], s["A"], s["B"], s["C"], s["bias"], s["workspace"])
    else:
        g.gemm_run(s["plan"], s["A"], s["B"], s["C"], s["bias"])
    return s["C"]


def exact(case, seed):
    c = case
    s = {k: v.to(torch.float32).to(torch.float64) for k, v in _inputs(case, seed).items()}
    if c["kind"] == "rope":
        cos, sin, h = s["cos"][None, :, None, :], s["sin"][None, :, None, :], c["head_dim"] // 2
        return [x * cos + torch.cat([-x[..., h:], x[..., :h]], dim=-1) * sin for x in (s["q"], s["k"])]
    if c["kind"] == "backward":
        return [s["dY"] @ s["W"], s["dY"].t().contiguous() @ s["X"]]
    t = torch.matmul(s["A"], s["B"] if c.get("b", "col") == "row" else s["B"].transpose(1, 2).contiguous())
    e = c.get("epilogue", "none")
    if "bias" in e:
        t += s["bias"]
    if e.endswith("relu"):
        t = t.clamp_min(0)
    elif e.endswith("gelu_erf"):
        t = 0.5 * t * (1 + torch.erf(t / math.sqrt(2)))
    elif e.endswith("gelu_tanh"):
        t = 0.5 * t * (1 + torch.tanh(math.sqrt(2 / math.pi) * (t + 0.044715 * t ** 3)))
    return t
