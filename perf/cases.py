"""Workloads of libcomfuse whose speed is tracked, through the public C entry points.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (operands, the output buffers, the argument block, the workspace),
`run` makes the call, `exact` gives the same outputs in 64 bits by plain torch.
The listed cases go from one short request to the largest batch of every
operator; `draw` gives further cases of the same ranges.
"""
import math

import torch

from paper_2608_03537_amd import comfuse as cf

EPS = 1e-5
BF16, F32 = torch.bfloat16, torch.float32


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # Latency of one small call: the fp32 post-norm block of 128 tokens.
        {"name": "postnorm_tiny_f32", "op": "postnorm", "dtype": "f32", "M": 128, "N": 256, "K": 256},
        # A short ragged batch through a BERT-base FFN-down projection with its post-norm.
        {"name": "postnorm_short", "op": "postnorm", "dtype": "bf16", "M": 333, "N": 768, "K": 3072},
        # BERT-base attention output + post-norm, 16 x 512 tokens.
        {"name": "postnorm_bert", "op": "postnorm", "dtype": "bf16", "M": 8192, "N": 768, "K": 768},
        # Scale, tanh softcap, softmax over 1024 classes: the smallest point of the batch sweep.
        {"name": "msts_2048", "op": "subgraph", "chain": "msts", "layout": "nk", "M": 2048, "N": 1024, "K": 1024},
        # LayerNorm, GELU, row amax, fp8 codes at the largest width and batch.
        {"name": "quant_chain_large", "op": "subgraph", "chain": "quant", "layout": "nk", "M": 16384, "N": 4096,
         "K": 4096},
        # The unfused pair with a K x N weight: a product, then RMSNorm over its rows.
        {"name": "gemm_then_norm_kn", "op": "pair", "layout": "kn", "M": 4096, "N": 4096, "K": 1024},
        # FFN block of the smaller model width on an odd number of rows.
        {"name": "ffn_ragged", "op": "ffn", "M": 3001, "d": 128, "N1": 256},
        # FFN block, 65536 tokens.
        {"name": "ffn_large", "op": "ffn", "M": 65536, "d": 256, "N1": 512},
        # Self-attention of 1000 tokens (not a multiple of a block), 12 heads of 64.
        {"name": "attention_ragged", "op": "attention", "B": 2, "H": 12, "Lq": 1000, "Lk": 1000, "d": 64},
        # Self-attention, 2048 tokens, 16 heads of 128.
        {"name": "attention_large", "op": "attention", "B": 4, "H": 16, "Lq": 2048, "Lk": 2048, "d": 128},
        # One decoding step: a single query per head against a long key list.
        {"name": "attention_decode", "op": "attention", "B": 8, "H": 16, "Lq": 1, "Lk": 4095, "d": 128},
        # DLRM bottom MLP 1024 -> 512 -> 128.
        {"name": "mlp_large", "op": "mlp", "M": 65536, "K": 1024, "N1": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the ranges of the listed ones."""
    op = rng.choice(["postnorm", "subgraph", "pair", "ffn", "attention", "attention", "mlp"])
    if op == "postnorm":
        n, k = rng.choice([(256, 256), (512, 512), (768, 768), (768, 3072), (1024, 1024), (1024, 4096),
                           (32 * rng.randint(4, 40), 16 * rng.randint(4, 100))])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        return {"op": op, "dtype": dtype, "M": _log(rng, 1, 32768 if dtype == "bf16" else 4096), "N": n, "K": k}
    if op == "subgraph":
        chain = rng.choice(["quant", "mbr", "mblr", "msts"])
        w = rng.choice([1024, 2048, 4096]) if chain == "quant" else 1024
        return {"op": op, "chain": chain, "layout": rng.choice(["nk", "nk", "kn"]),
                "M": _log(rng, 16, 16384 if chain == "quant" else 32768), "N": w, "K": w}
    if op == "pair":
        return {"op": op, "layout": rng.choice(["nk", "kn"]), "M": _log(rng, 16, 16384),
                "N": rng.choice([768, 1024, 2048, 4096]), "K": rng.choice([768, 1024, 2048, 4096])}
    if op == "ffn":
        n1, d = rng.choice([(512, 256), (256, 256), (256, 128), (128, 64)])
        return {"op": op, "M": _log(rng, 1, 65536), "d": d, "N1": n1}
    if op == "mlp":
        return {"op": op, "M": _log(rng, 1, 65536), "K": rng.choice([256, 512, 1024]),
                "N1": rng.choice([256, 512, 1024])}
    h, d = rng.choice([(8, 64), (12, 64), (16, 64), (16, 128)])
    form = rng.choice(["self", "cross", "decode"])
    if form == "self":
        lq = lk = _log(rng, 32, 4096)
        b = _log(rng, 1, max(1, min(16, (1 << 24) // (lq * lq))))
    elif form == "cross":                     # many target rows against a short source
        lq, lk, b = _log(rng, 256, 4096), _log(rng, 64, 512), _log(rng, 1, 8)
    else:
        lq, lk, b = rng.choice([1, 1, 2, 4, 16]), _log(rng, 64, 8192), _log(rng, 1, 16)
    return {"op": op, "B": b, "H": h, "Lq": lq, "Lk": lk, "d": d}


# ---------------------------------------------------------------- inputs
class _Draw:
    """Normal tensors on the GPU from one seed, in call order."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def __call__(self, shape, std=1.0, dtype=BF16, mean=0.0):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=F32)
        return (t * std + mean).to(dtype)


def _operands(case, seed):
    """The tensors of a case: weights at variance 1/K, small biases, a scale near 1."""
    r, op = _Draw(seed), case["op"]
    if op == "postnorm":
        M, N, K = case["M"], case["N"], case["K"]
        dt = F32 if case["dtype"] == "f32" else BF16
        return dict(X=r((M, K), dtype=dt), W=r((N, K), K ** -0.5, dt), b=r((N,), 0.02, F32), R=r((M, N), dtype=dt),
                    g=r((N,), 0.02, F32, 1.0), be=r((N,), 0.02, F32))
    if op in ("subgraph", "pair"):
        M, N, K = case["M"], case["N"], case["K"]
        t = dict(X=r((M, K)), W=r((N, K) if case["layout"] == "nk" else (K, N), K ** -0.5), b=r((N,), 0.02, F32))
        if op == "pair" or case["chain"] in ("mbr", "mblr"):
            t["g"] = r((N,), 0.02, F32, 1.0)
        if op == "subgraph" and case["chain"] == "quant":
            t["R"] = r((M, N))
        return t
    if op == "ffn":
        M, d, n = case["M"], case["d"], case["N1"]
        return dict(X=r((M, d)), W1=r((n, d), d ** -0.5), b1=r((n,), 0.02, F32), W2=r((d, n), n ** -0.5),
                    b2=r((d,), 0.02, F32))
    if op == "mlp":
        M, k, n = case["M"], case["K"], case["N1"]
        return dict(X=r((M, k)), W1=r((n, k), k ** -0.5), b1=r((n,), 0.02, F32), W2=r((128, n), n ** -0.5),
                    b2=r((128,), 0.02, F32))
    B, H, d = case["B"], case["H"], case["d"]
    return dict(Q=r((B, H, case["Lq"], d)), K=r((B, H, case["Lk"], d)), V=r((B, H, case["Lk"], d)))


def _b2b(**kw):
    a = cf.B2BArgs()
    a.struct_size = cf.C.sizeof(cf.B2BArgs)
    a.dtype, a.batch, a.mid_scale = cf.CF_BF16, 1, 1.0
    for k, v in kw.items():
        setattr(a, k, v.data_ptr() if isinstance(v, torch.Tensor) else v)
    return a


def _layout(case):
    return cf.CF_LAYOUT_NK if case.get("layout", "nk") == "nk" else cf.CF_LAYOUT_KN


def _store(t):
    return dict(kind=cf.CF_N_STORE, out=t, ld=t.stride(0), dtype=cf.CF_BF16)


def prepare(case, seed):
    t, op = _operands(case, seed), case["op"]
    s = {"op": op, "t": t, "stream": torch.cuda.current_stream().cuda_stream, "ws": None}

    def empty(*shape, dtype=BF16):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if op == "postnorm":
        y = empty(case["M"], case["N"], dtype=t["X"].dtype)
        s["args"] = cf.postnorm_args(t["X"], t["W"], t["b"], t["R"], t["g"], t["be"], y, eps=EPS)
        s["ws"] = cf.workspace(cf.cf_gemm_postnorm_workspace(s["args"]), "cuda")
        s["out"] = [y]
    elif op == "subgraph":
        M, N = case["M"], case["N"]
        y = empty(M, N)
        s["out"] = [y]
        nodes = {"quant": lambda: [dict(kind=cf.CF_N_BIAS, v0=t["b"]),
                                   dict(kind=cf.CF_N_RESIDUAL, ld=N, dtype=cf.CF_BF16, **{"in": t["R"]}),
                                   dict(kind=cf.CF_N_LAYERNORM, f0=EPS), dict(kind=cf.CF_N_GELU), _store(y),
                                   dict(kind=cf.CF_N_ROWAMAX_QUANT, out=s["out"][1], out2=s["out"][2], ld=N, f0=448.0)],
                 "mbr": lambda: [dict(kind=cf.CF_N_BIAS, v0=t["b"]),
                                 dict(kind=cf.CF_N_RMSNORM, v0=t["g"], f0=EPS), _store(y)],
                 "mblr": lambda: [dict(kind=cf.CF_N_BIAS, v0=t["b"]),
                                  dict(kind=cf.CF_N_LAYERNORM, v0=t["g"], f0=EPS), dict(kind=cf.CF_N_RELU), _store(y)],
                 "msts": lambda: [dict(kind=cf.CF_N_SCALE, f0=8.0), dict(kind=cf.CF_N_SOFTCAP, f0=10.0),
                                  dict(kind=cf.CF_N_SOFTMAX), _store(y)]}
        if case["chain"] == "quant":
            s["out"] += [empty(M, dtype=F32), empty(M, N, dtype=torch.uint8)]
        s["nodes"] = cf.make_nodes(nodes[case["chain"]]())
        s["args"] = cf.subgraph_args(t["X"], t["W"], s["nodes"], w_layout=_layout(case))
        s["ws"] = cf.workspace(cf.cf_gemm_subgraph_workspace(s["args"]), "cuda")
    elif op == "pair":
        M, N, K = case["M"], case["N"], case["K"]
        p, y = empty(M, N), empty(M, N)
        s["out"] = [p, y]
        s["nodes"] = cf.make_nodes([dict(kind=cf.CF_N_BIAS, v0=t["b"]),
                                    dict(kind=cf.CF_N_RMSNORM, v0=t["g"], f0=EPS), _store(y)])
        s["gemm"] = (1, M, N, K, cf.CF_BF16, cf.CF_BF16, t["X"].data_ptr(), K, 0, t["W"].data_ptr(),
                     t["W"].stride(0), 0, _layout(case), None, 1.0, p.data_ptr(), N, 0, s["stream"])
        s["rows"] = (1, M, N, cf.CF_BF16, p.data_ptr(), N, 0, s["nodes"], len(s["nodes"]), s["stream"])
    elif op == "ffn":
        M, d, n = case["M"], case["d"], case["N1"]
        o = empty(M, d)
        s["out"] = [o]
        s["args"] = _b2b(M=M, K=d, N1=n, N2=d, X=t["X"], ldx=d, W1=t["W1"], ldw1=d, w1_layout=cf.CF_LAYOUT_NK,
                         b1=t["b1"], mid=cf.CF_MID_GELU_BIAS, W2=t["W2"], ldw2=n, w2_layout=cf.CF_LAYOUT_NK,
                         out=cf.CF_OUT_BIAS_RESIDUAL_LN, b2=t["b2"], R=t["X"], ldr=d, eps=EPS, O=o, ldo=d)
    elif op == "mlp":
        M, k, n = case["M"], case["K"], case["N1"]
        o = empty(M, 128)
        s["out"] = [o]
        s["args"] = _b2b(M=M, K=k, N1=n, N2=128, X=t["X"], ldx=k, W1=t["W1"], ldw1=k, w1_layout=cf.CF_LAYOUT_NK,
                         b1=t["b1"], mid=cf.CF_MID_RELU_BIAS, W2=t["W2"], ldw2=n, w2_layout=cf.CF_LAYOUT_NK,
                         out=cf.CF_OUT_STORE, b2=t["b2"], O=o, ldo=128)
        s["ws"] = cf.workspace(cf.cf_b2bgemm_workspace(s["args"]), "cuda", kind="b2b")
    else:
        B, H, lq, lk, d = (case[k] for k in ("B", "H", "Lq", "Lk", "d"))
        o = empty(B, H, lq, d)
        s["out"] = [o]
        s["args"] = _b2b(batch=B * H, M=lq, K=d, N1=lk, N2=d, X=t["Q"], ldx=d, sx=lq * d, W1=t["K"], ldw1=d,
                         sw1=lk * d, w1_layout=cf.CF_LAYOUT_NK, mid=cf.CF_MID_SOFTMAX, mid_scale=d ** -0.5,
                         W2=t["V"], ldw2=d, sw2=lk * d, w2_layout=cf.CF_LAYOUT_KN, out=cf.CF_OUT_STORE, O=o, ldo=d,
                         so=lq * d)
        s["ws"] = cf.workspace(cf.cf_b2bgemm_workspace(s["args"]), "cuda", kind="b2b")
    ws = s["ws"]
    s["ws_arg"] = (None, 0) if ws is None else (ws.data_ptr(), ws.numel())
    return s


# ---------------------------------------------------------------- the call
def _ok(status):
    if status != 0:
        raise cf.CfError(status, cf.cf_last_error())


def run(s):
    op = s["op"]
    if op == "postnorm":
        _ok(cf.cf_gemm_postnorm(s["args"], *s["ws_arg"], s["stream"]))
    elif op == "subgraph":
        _ok(cf.cf_gemm_subgraph(s["args"], *s["ws_arg"], s["stream"]))
    elif op == "pair":
        _ok(cf.cf_gemm(*s["gemm"]))
        _ok(cf.cf_rowop(*s["rows"]))
    else:
        _ok(cf.cf_b2bgemm(s["args"], *s["ws_arg"], s["stream"]))
    return s["out"]


def work(case):
    """Bytes with each operand read once and each output written once; the contractions' operations."""
    op = case["op"]
    if op in ("postnorm", "subgraph", "pair"):
        M, N, K = case["M"], case["N"], case["K"]
        e = 4 if case.get("dtype") == "f32" else 2
        mn = {"postnorm": 2 * e, "pair": 3 * e}.get(op)          # R, Y; the pair writes P, reads it, writes Y
        if op == "subgraph":
            mn = 5 if case["chain"] == "quant" else 2             # R, Z, codes; Y
        vec = 4 * N * (3 if op == "postnorm" else 2) + (4 * M if case.get("chain") == "quant" else 0)
        return {"bytes": e * (M * K + N * K) + mn * M * N + vec, "flops": 2 * M * N * K}
    if op == "ffn":
        M, d, n = case["M"], case["d"], case["N1"]
        return {"bytes": 2 * (2 * M * d + 2 * d * n) + 4 * (n + d), "flops": 4 * M * d * n}
    if op == "mlp":
        M, k, n = case["M"], case["K"], case["N1"]
        return {"bytes": 2 * (M * (k + 128) + k * n + 128 * n) + 4 * (n + 128), "flops": 2 * M * n * (k + 128)}
    bh, lq, lk, d = case["B"] * case["H"], case["Lq"], case["Lk"], case["d"]
    return {"bytes": 4 * bh * d * (lq + lk), "flops": 4 * bh * lq * lk * d}


def tolerance(case):
    """About four times the error against `exact` (bf16 outputs: half an ulp, 1.7e-3 in the 2-norm; the rounding of
    the intermediate to bf16 adds a little in the back-to-back products; fp32: sums of K terms)."""
    if case.get("dtype") == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    if case.get("chain") == "quant":
        return {"rel": 7e-3, "max": 3e-2, "differ": 1e-3}
    if case["op"] in ("ffn", "mlp", "attention"):
        return {"rel": 1e-2, "max": 5e-2}
    return {"rel": 7e-3, "max": 3e-2}


# ---------------------------------------------------------------- 64 bits
def exact(case, seed):
    t = {k: v.double() for k, v in _operands(case, seed).items()}
    op = case["op"]

    def layernorm(x):
        x = x - x.mean(1, keepdim=True)
        return x / torch.sqrt(x.square().mean(1, keepdim=True) + EPS)

    def rmsnorm(x):
        return x / torch.sqrt(x.square().mean(1, keepdim=True) + EPS)

    def gelu(x):
        return x * 0.5 * (1.0 + torch.erf(x * math.sqrt(0.5)))

    if op in ("postnorm", "subgraph", "pair"):
        p = t["X"] @ (t["W"].t() if case.get("layout", "nk") == "nk" else t["W"])
        if op == "postnorm":
            return [layernorm(p + t["b"] + t["R"]) * t["g"] + t["be"]]
        if op == "pair":   # the row operator reads the product as it was stored
            return [p, rmsnorm(p.to(BF16).double() + t["b"]) * t["g"]]
        if case["chain"] == "quant":
            z = gelu(layernorm(p + t["b"] + t["R"]))
            return [z, z.abs().amax(1) / 448.0, None]
        if case["chain"] == "mbr":
            return [rmsnorm(p + t["b"]) * t["g"]]
        if case["chain"] == "mblr":
            return [torch.relu(layernorm(p + t["b"]) * t["g"])]
        return [torch.softmax(10.0 * torch.tanh(p * 8.0 / 10.0), 1)]
    if op == "ffn":
        return [layernorm(gelu(t["X"] @ t["W1"].t() + t["b1"]) @ t["W2"].t() + t["b2"] + t["X"])]
    if op == "mlp":
        return [torch.relu(t["X"] @ t["W1"].t() + t["b1"]) @ t["W2"].t() + t["b2"]]
    q, k, v = (t[n].flatten(0, 1) for n in ("Q", "K", "V"))
    o = torch.empty_like(q)
    for h in range(q.shape[0]):
        o[h] = torch.softmax(q[h] @ k[h].t() * case["d"] ** -0.5, 1) @ v[h]
    return [o.view(t["Q"].shape)]
