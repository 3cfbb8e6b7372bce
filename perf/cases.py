"""The work this framework is timed on: single layers through pw_op_*, compiled functions and whole steps.

Families: chains of trivial compiled functions (dispatch), the feed-forward block, attention in its three roles,
LayerNorm, the LM head with its loss, the embedding tables, a pipeline stage and a whole LM train step.  Every layer
is taken forward and backward, as a training program takes it.  Sizes are those of the repository's workloads and
tests (model widths 256 to 2048, sequences of 80 to 2048 positions, vocabularies of 1024 to 32768) and ragged ones
between them.
"""
import math

import numpy as np
import torch

from paper_2203_12533_amd import binding as pwb
from paper_2203_12533_amd import inputs as I

_DT = {"f32": pwb.PW_F32, "bf16": pwb.PW_BF16}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_context = None


def _ctx():
    """One context per program, as in any program that uses the library."""
    global _context
    if _context is None:
        _context = pwb.Context(0)
    return _context


# ---- the cases -------------------------------------------------------------------------------------------------

def listed():
    return [
        # the dispatch micro-benchmark: a program of 32 trivial functions on a small buffer, result fetched
        {"name": "chain_32", "family": "chain", "length": 32, "n": 128, "mode": "stream"},
        # the feed-forward block of the measured 12-layer LM, all of its tokens
        {"name": "ffn_8192x2048", "family": "ffn", "dtype": "bf16", "tokens": 8192, "d": 2048, "ff": 8192},
        # a small model's feed-forward block: a batch that fits no tile
        {"name": "ffn_1000x768", "family": "ffn", "dtype": "bf16", "tokens": 1000, "d": 768, "ff": 3072},
        # the same in single precision (the configuration that is checked digit by digit)
        {"name": "ffn_f32_512x256", "family": "ffn", "dtype": "f32", "tokens": 512, "d": 256, "ff": 1024},
        # causal self-attention of the measured LM
        {"name": "attn_causal_128", "family": "attention", "dtype": "bf16", "role": "causal", "batch": 8, "tq": 1024,
         "tk": 1024, "heads": 16, "hd": 128},
        # causal self-attention at the other head width, a sequence that fits no tile
        {"name": "attn_causal_64", "family": "attention", "dtype": "bf16", "role": "causal", "batch": 4, "tq": 1000,
         "tk": 1000, "heads": 12, "hd": 64},
        # a decoder's attention over the encoder output, target and source of different ragged lengths
        {"name": "attn_cross_64", "family": "attention", "dtype": "bf16", "role": "cross", "batch": 4, "tq": 333,
         "tk": 520, "heads": 8, "hd": 64},
        # LayerNorm of the measured LM's residual stream
        {"name": "layernorm_8192x2048", "family": "layernorm", "dtype": "bf16", "rows": 8192, "d": 2048},
        # LM head and loss of the measured LM
        {"name": "head_8192x32768", "family": "head", "dtype": "bf16", "batch": 8, "seq": 1024, "d": 2048, "vocab": 32768},
        # its embedding tables
        {"name": "embedding_8192", "family": "embedding", "batch": 8, "seq": 1024, "d": 2048, "vocab": 32768},
        # one layer of the measured LM as a pipeline stage: two micro-batches forward, then backward, then the update
        {"name": "stage_2x2048", "family": "stage", "dtype": "bf16", "batch": 2, "seq": 1024, "d": 2048, "heads": 16,
         "ff": 8192, "microbatches": 2},
        # the small fp32 workload as a whole train step, all gradients read back as a checking program reads them
        {"name": "lm_step_f32", "family": "lm", "dtype": "f32", "layers": 2, "batch": 4, "seq": 128, "d": 256, "heads": 4,
         "ff": 1024, "vocab": 1024, "optimizer": "sgd"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, m):
    return max(m, _log(rng, lo, hi) // m * m)


def draw(rng):
    family = rng.choice(["chain", "ffn", "ffn", "attention", "attention", "attention", "layernorm", "head", "embedding",
                         "stage", "lm"])
    if family == "chain":
        return {"family": family, "length": _log(rng, 1, 128), "n": _log(rng, 1, 4096),
                "mode": rng.choice(["stream", "graph"])}
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if family == "ffn":
        if dtype == "f32":
            return {"family": family, "dtype": dtype, "tokens": _log(rng, 64, 1024), "d": _mult(rng, 128, 512, 64),
                    "ff": _mult(rng, 256, 2048, 64)}
        return {"family": family, "dtype": dtype, "tokens": _mult(rng, 64, 8192, 8), "d": _mult(rng, 256, 2048, 64),
                "ff": _mult(rng, 1024, 8192, 64)}
    if family == "attention":
        role = rng.choice(["causal", "self", "cross"])
        tq = _log(rng, 40, 2048 if dtype == "bf16" else 256)
        tk = _log(rng, 40, 2048 if dtype == "bf16" else 256) if role == "cross" else tq
        heads = _log(rng, 2, 16)
        most = max(1, (1 << 27 if dtype == "bf16" else 1 << 21) // (tq * tk * heads))
        return {"family": family, "dtype": dtype, "role": role, "batch": min(_log(rng, 1, 8), most), "tq": tq, "tk": tk,
                "heads": heads, "hd": rng.choice([64, 128])}
    if family == "layernorm":
        rows = _log(rng, 8, 8192)
        return {"family": family, "dtype": dtype, "rows": rows, "d": _mult(rng, 256, min(8192, (1 << 24) // rows), 4)}
    if family == "head":
        return {"family": family, "dtype": "bf16", "batch": 8, "seq": _log(rng, 16, 1024), "d": _mult(rng, 256, 2048, 64),
                "vocab": _mult(rng, 1024, 32768, 8)}
    if family == "embedding":
        return {"family": family, "batch": _log(rng, 1, 8), "seq": _log(rng, 16, 1024), "d": _mult(rng, 256, 2048, 4),
                "vocab": _log(rng, 1024, 32768)}
    hd = rng.choice([64, 128])
    if family == "stage":
        heads = _log(rng, 2, 2048 // hd)
        return {"family": family, "dtype": "bf16", "batch": _log(rng, 1, 2), "seq": _mult(rng, 64, 1024, 8),
                "d": heads * hd, "heads": heads, "ff": _mult(rng, 1024, 8192, 64), "microbatches": 2}
    heads = _log(rng, 2, 512 // hd)
    return {"family": family, "dtype": dtype, "layers": rng.choice([1, 2]), "batch": _log(rng, 1, 4),
            "seq": _mult(rng, 64, 256, 8), "d": heads * hd, "heads": heads, "ff": _mult(rng, 256, 2048, 64),
            "vocab": _mult(rng, 512, 2048, 8), "optimizer": "sgd" if dtype == "f32" else "adam"}


# ---- inputs ----------------------------------------------------------------------------------------------------

class _Draw:
    """Seeded normals and token ids on the GPU; the order of the calls is part of the recipe."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) * 7919 + 17)

    def normal(self, *shape, std=1.0, dtype=torch.float32, mean=0.0):
        t = torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)
        return t.mul_(std).add_(mean).to(dtype)

    def ids(self, *shape, vocab):
        return torch.randint(0, vocab, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _ffn_inputs(c, seed):
    r, t = _Draw(seed), _TORCH[c["dtype"]]
    n, d, f = c["tokens"], c["d"], c["ff"]
    return {"a": r.normal(n, d, dtype=t), "w1": r.normal(d, f, std=0.02, dtype=t), "b1": r.normal(f, std=0.02),
            "w2": r.normal(f, d, std=0.02, dtype=t), "b2": r.normal(d, std=0.02), "x": r.normal(n, d),
            "dy": r.normal(n, d, std=1e-2, dtype=t)}


def _attention_inputs(c, seed):
    r, t = _Draw(seed), _TORCH[c["dtype"]]
    b, tq, tk, d = c["batch"], c["tq"], c["tk"], c["heads"] * c["hd"]
    s = {"dout": r.normal(b * tq, d, std=1e-2, dtype=t)}
    if c["role"] == "cross":
        s["q"], s["kv"] = r.normal(b * tq, d, dtype=t), r.normal(b * tk, 2 * d, dtype=t)
    else:
        s["qkv"] = r.normal(b * tq, 3 * d, dtype=t)
    return s


def _layernorm_inputs(c, seed):
    r, n, d = _Draw(seed), c["rows"], c["d"]
    return {"x": r.normal(n, d, mean=0.1), "g": r.normal(d, std=0.1, mean=1.0), "b": r.normal(d, std=0.1),
            "dy": r.normal(n, d, std=1e-2, dtype=_TORCH[c["dtype"]]), "dres": r.normal(n, d, std=1e-2)}


def _head_inputs(c, seed):
    r, t, n = _Draw(seed), _TORCH[c["dtype"]], c["batch"] * c["seq"]
    return {"y": r.normal(n, c["d"], dtype=t), "wh": r.normal(c["d"], c["vocab"], std=0.02, dtype=t),
            "tokens": r.ids(c["batch"], c["seq"] + 1, vocab=c["vocab"])}


def _embedding_inputs(c, seed):
    r = _Draw(seed)
    return {"wte": r.normal(c["vocab"], c["d"], std=0.02), "wpe": r.normal(c["seq"], c["d"], std=0.02),
            "tokens": r.ids(c["batch"], c["seq"] + 1, vocab=c["vocab"]),
            "dx": r.normal(c["batch"] * c["seq"], c["d"], std=1e-2)}


def _lm_config(c):
    stage = c["family"] == "stage"
    return I.LMConfig(1 if stage else c["layers"], c["d"], c["heads"], c["ff"], 0 if stage else c["vocab"], c["seq"],
                      c["batch"], bf16=c["dtype"] == "bf16", optimizer="adam" if stage else c["optimizer"],
                      lr=1e-2 if c.get("optimizer") == "sgd" else 1e-4, has_embed=not stage, has_head=not stage,
                      n_microbatch=c.get("microbatches", 1))


def _params(c, r):
    """Random biases and gains as well: zeros and ones would hide them.  Values a bf16 model can start from."""
    out = {}
    for name, shape, kind in I.param_shapes(_lm_config(c)):
        t = r.normal(*shape, std=0.02, mean=1.0 if kind == "gain" else 0.0)
        out[name] = t.to(torch.bfloat16).float() if c["dtype"] == "bf16" else t
    return out


def _stage_inputs(c, seed):
    r, n = _Draw(seed), c["batch"] * c["seq"]
    p = _params(c, r)
    low = lambda t: t.to(torch.bfloat16).float()  # noqa: E731  (activations cross a stage boundary as such values)
    xs = [low(r.normal(n, c["d"])) for _ in range(c["microbatches"])]
    dys = [low(r.normal(n, c["d"], std=1e-2)) for _ in range(c["microbatches"])]
    return p, xs, dys


def _lm_inputs(c, seed):
    r = _Draw(seed)
    return _params(c, r), r.ids(c["batch"], c["seq"] + 1, vocab=c["vocab"])


class _OwnedModel:
    """A model whose device memory goes when its last user does."""

    def __init__(self, cfg, params):
        self.m = _ctx().model(cfg)
        torch.cuda.synchronize()
        for name, t in params.items():
            self.m.import_device(pwb.PW_PARAMS, name, t.data_ptr())

    def __del__(self):
        self.m.close()


class _Futures:
    """Handles a program holds on to, given back with their holder."""

    def __init__(self, handles=()):
        self.handles = list(handles)

    def replace(self, handles):
        old, self.handles = self.handles, list(handles)
        for f in old:
            _ctx().future_release(f)

    def __del__(self):
        self.replace([])


class _DeviceArray:
    """A future's buffer as something torch can look at without a copy."""

    def __init__(self, ptr, shape):
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": tuple(shape), "typestr": "<f4", "version": 2}


def prepare(case, seed):
    c, ctx, fam = case, _ctx(), case["family"]
    s = {"case": dict(case)}
    if fam == "chain":
        x = _Draw(seed).normal(c["n"]).cpu().numpy()
        s["fns"] = [ctx.compile_scalar_fn(pwb.PW_FN_ADD_CONST, c["n"], 1.0)] * c["length"]
        s["in"] = _Futures([ctx.future_from_host(x)])
        s["mode"] = {"stream": pwb.PW_STREAM, "graph": pwb.PW_GRAPH}[c["mode"]]
        ctx.synchronize()
        return s
    new = lambda *shape, dtype=torch.float32: torch.empty(*shape, dtype=dtype, device="cuda")  # noqa: E731
    t = _TORCH.get(c.get("dtype"))
    if fam == "ffn":
        s.update(_ffn_inputs(c, seed))
        n, d, f = c["tokens"], c["d"], c["ff"]
        s.update(u=new(n, f, dtype=t), h=new(n, f, dtype=t), y=new(n, d), du=new(n, f, dtype=t), da=new(n, d, dtype=t),
                 dw1=new(d, f), dw2=new(f, d), db1=new(f), ws=new(pwb.lib().pw_colsum_ws_floats(n, f)))
    elif fam == "attention":
        s.update(_attention_inputs(c, seed))
        b, tq, tk, h, d = c["batch"], c["tq"], c["tk"], c["heads"], c["heads"] * c["hd"]
        s.update(o=new(b * tq, d, dtype=t), lse=new(b, h, tq), delta=new(b, h, tq))
        if c["role"] == "causal":
            s["dqkv"] = new(b * tq, 3 * d, dtype=t)
        else:
            s["o_lo"] = new(b * tq, d, dtype=t)
            if c["role"] == "self":
                s["dqkv"] = new(b * tq, 3 * d, dtype=t)
            else:
                s["dq"], s["dkv"] = new(b * tq, d, dtype=t), new(b * tk, 2 * d, dtype=t)
    elif fam == "layernorm":
        s.update(_layernorm_inputs(c, seed))
        n, d = c["rows"], c["d"]
        s.update(y=new(n, d, dtype=t), mean=new(n), rstd=new(n), dx=new(n, d), dx_lp=new(n, d, dtype=t), dg=new(d),
                 db=new(d), dsum=new(d), ws=new(pwb.lib().pw_layernorm_bwd_ws_floats(n, d)))
    elif fam == "head":
        s.update(_head_inputs(c, seed))
        n = c["batch"] * c["seq"]
        s.update(z=new(n, c["vocab"], dtype=t), loss=new(1), row_loss=new(n), dy=new(n, c["d"], dtype=t),
                 dwh=new(c["d"], c["vocab"]))
    elif fam == "embedding":
        s.update(_embedding_inputs(c, seed))
        s.update(x=new(c["batch"] * c["seq"], c["d"]), dwte=new(c["vocab"], c["d"]), dwpe=new(c["seq"], c["d"]))
    elif fam == "stage":
        p, s["xs"], s["dys"] = _stage_inputs(c, seed)
        s["model"] = _OwnedModel(_lm_config(c), p)
        m, shape, mbs = s["model"].m, (c["batch"] * c["seq"], c["d"]), range(c["microbatches"])
        s["fwd"] = [m.compile_stage(pwb.PW_FN_STAGE_FWD, i) for i in mbs]
        s["bwd"] = [m.compile_stage(pwb.PW_FN_STAGE_BWD, i) for i in mbs]
        s["in"] = _Futures([ctx.future_wrap_device(a.data_ptr(), pwb.PW_F32, shape) for a in s["xs"] + s["dys"]])
        s["out"] = _Futures()
        s["shape"] = shape
    else:
        p, tok = _lm_inputs(c, seed)
        s["model"] = _OwnedModel(_lm_config(c), p)
        s["step"] = s["model"].m.compile_train_step()
        s["tok"] = tok
        s["in"] = _Futures([ctx.future_wrap_device(tok.data_ptr(), pwb.PW_I32, tuple(tok.shape))])
    torch.cuda.synchronize()
    return s


# ---- one pass --------------------------------------------------------------------------------------------------

def _run_chain(s, c, ctx):
    (f,) = ctx.chain(s["fns"], s["in"].handles, 1, s["mode"])
    out = ctx.await_(f)
    ctx.future_release(f)
    return out


def _run_ffn(s, c, ctx):
    p = lambda k: s[k].data_ptr()  # noqa: E731
    n, d, f, dt = c["tokens"], c["d"], c["ff"], _DT[c["dtype"]]
    k = dict(dtype=dt, accumulate=0)
    ctx.gemm(a_kmajor=0, b_kmajor=1, M=n, N=f, K=d, lda=d, ldb=f, ldc=f, epilogue=pwb.PW_EPI_BIAS_GELU, out_dtype=dt,
             A=p("a"), B=p("w1"), bias=p("b1"), C=p("u"), C2=p("h"), **k)
    ctx.gemm(a_kmajor=0, b_kmajor=1, M=n, N=d, K=f, lda=f, ldb=d, ldc=d, epilogue=pwb.PW_EPI_BIAS_RESIDUAL,
             out_dtype=pwb.PW_F32, A=p("h"), B=p("w2"), bias=p("b2"), aux=p("x"), C=p("y"), **k)
    ctx.gemm(a_kmajor=0, b_kmajor=0, M=n, N=f, K=d, lda=d, ldb=d, ldc=f, epilogue=pwb.PW_EPI_GELU_BWD, out_dtype=dt,
             A=p("dy"), B=p("w2"), aux=p("u"), C=p("du"), **k)
    ctx.gemm(a_kmajor=0, b_kmajor=0, M=n, N=d, K=f, lda=f, ldb=f, ldc=d, epilogue=pwb.PW_EPI_STORE, out_dtype=dt,
             A=p("du"), B=p("w1"), C=p("da"), **k)
    ctx.gemm(a_kmajor=1, b_kmajor=1, M=f, N=d, K=n, lda=f, ldb=d, ldc=d, epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32,
             A=p("h"), B=p("dy"), C=p("dw2"), **k)
    ctx.gemm(a_kmajor=1, b_kmajor=1, M=d, N=f, K=n, lda=d, ldb=f, ldc=f, epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32,
             A=p("a"), B=p("du"), C=p("dw1"), **k)
    ctx.op("colsum", dt, p("du"), p("db1"), p("ws"), n, f, 0)
    return {i: s[i] for i in ("h", "y", "da", "dw1", "dw2", "db1")}


def _run_attention(s, c, ctx):
    p = lambda k: s[k].data_ptr()  # noqa: E731
    b, tq, tk, h, hd, dt = c["batch"], c["tq"], c["tk"], c["heads"], c["hd"], _DT[c["dtype"]]
    d, es = h * hd, s["o"].element_size()
    if c["role"] == "causal":
        ctx.op("attention_fwd", dt, p("qkv"), p("o"), p("lse"), b, tq, h, hd)
        ctx.op("attention_bwd", dt, p("qkv"), p("o"), p("dout"), p("lse"), p("delta"), p("dqkv"), b, tq, h, hd)
        return {i: s[i] for i in ("o", "lse", "dqkv")}
    if c["role"] == "self":
        q, kk, v, ldq, ldkv = p("qkv"), p("qkv") + d * es, p("qkv") + 2 * d * es, 3 * d, 3 * d
        dq, dk, dv = p("dqkv"), p("dqkv") + d * es, p("dqkv") + 2 * d * es
    else:
        q, kk, v, ldq, ldkv = p("q"), p("kv"), p("kv") + d * es, d, 2 * d
        dq, dk, dv = p("dq"), p("dkv"), p("dkv") + d * es
    a = pwb.MhaArgs(dt, q, kk, v, ldq, ldkv, b, tq, tk, h, hd, 0)
    ctx.mha_fwd(a, p("o"), p("lse"), p("o_lo"))
    ctx.mha_bwd(a, p("o"), p("dout"), p("lse"), p("delta"), dq, ldq, dk, dv, ldkv, p("o_lo"))
    return {i: s[i] for i in (("o", "lse", "dqkv") if c["role"] == "self" else ("o", "lse", "dq", "dkv"))}


def _run_layernorm(s, c, ctx):
    p = lambda k: s[k].data_ptr()  # noqa: E731
    n, d, dt = c["rows"], c["d"], _DT[c["dtype"]]
    ctx.op("layernorm_fwd", dt, p("x"), p("g"), p("b"), p("y"), p("mean"), p("rstd"), n, d)
    ctx.op("layernorm_bwd", dt, p("dy"), p("x"), p("g"), p("mean"), p("rstd"), p("dres"), p("dx"), p("dx_lp"), p("dg"),
           p("db"), p("dsum"), p("ws"), n, d, 0)
    names = ("y", "mean", "rstd", "dx", "dg", "db", "dsum")
    return {i: s[i] for i in (names + ("dx_lp",) if c["dtype"] == "bf16" else names)}


def _run_head(s, c, ctx):
    p = lambda k: s[k].data_ptr()  # noqa: E731
    n, d, v, dt = c["batch"] * c["seq"], c["d"], c["vocab"], _DT[c["dtype"]]
    k = dict(dtype=dt, accumulate=0, epilogue=pwb.PW_EPI_STORE)
    ctx.gemm(a_kmajor=0, b_kmajor=1, M=n, N=v, K=d, lda=d, ldb=v, ldc=v, out_dtype=dt, A=p("y"), B=p("wh"), C=p("z"), **k)
    ctx.op("softmax_xent", dt, p("z"), p("tokens"), p("loss"), p("row_loss"), c["batch"], c["seq"], v)
    ctx.gemm(a_kmajor=0, b_kmajor=0, M=n, N=d, K=v, lda=v, ldb=v, ldc=d, out_dtype=dt, A=p("z"), B=p("wh"), C=p("dy"), **k)
    ctx.gemm(a_kmajor=1, b_kmajor=1, M=d, N=v, K=n, lda=d, ldb=v, ldc=v, out_dtype=pwb.PW_F32, A=p("y"), B=p("z"),
             C=p("dwh"), **k)
    return {i: s[i] for i in ("loss", "row_loss", "z", "dy", "dwh")}


def _run_embedding(s, c, ctx):
    p = lambda k: s[k].data_ptr()  # noqa: E731
    dims = (c["batch"], c["seq"], c["d"], c["vocab"])
    ctx.op("embedding_fwd", p("tokens"), p("wte"), p("wpe"), p("x"), *dims)
    ctx.op("embedding_bwd", p("tokens"), p("dx"), p("dwte"), p("dwpe"), *dims)
    return {i: s[i] for i in ("x", "dwte", "dwpe")}


# What a program that watches a stage reads back every step: the gradients of its vectors.
_STAGE_READ = ("l0.ln1_g", "l0.bqkv", "l0.bo", "l0.b1")


def _run_stage(s, c, ctx):
    m, n_mb = s["model"].m, c["microbatches"]
    f = s["in"].handles
    m.zero_grads()
    ys = [ctx.run_fn(s["fwd"][i], [f[i]])[0] for i in range(n_mb)]
    dxs = [ctx.run_fn(s["bwd"][i], [f[n_mb + i]])[0] for i in reversed(range(n_mb))][::-1]
    m.apply_optimizer()
    s["out"].replace(ys + dxs)
    view = lambda h: torch.as_tensor(_DeviceArray(ctx.future_device_ptr(h), s["shape"]), device="cuda")  # noqa: E731
    return {"y": [view(h) for h in ys], "dx": [view(h) for h in dxs],
            "grads": {k: m.export(pwb.PW_GRADS, k) for k in _STAGE_READ}}


def _run_lm(s, c, ctx):
    m = s["model"].m
    f = ctx.train_step(s["step"], s["in"].handles[0])
    loss = ctx.await_(f)
    ctx.future_release(f)
    return {"loss": loss, "dlogits": m.export_activation("dlogits", c["batch"] * c["seq"] * c["vocab"]),
            "grads": {k: m.export(pwb.PW_GRADS, k) for k in m.names}}


_RUN = {"chain": _run_chain, "ffn": _run_ffn, "attention": _run_attention, "layernorm": _run_layernorm, "head": _run_head,
        "embedding": _run_embedding, "stage": _run_stage, "lm": _run_lm}


def run(state):
    c = state["case"]
    return _RUN[c["family"]](state, c, _ctx())


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def _layer_flops(n, t, d, f):
    """Forward and backward of one layer over n tokens in sequences of t, causal attention at half of t^2."""
    return 6.0 * n * (4 * d * d + 2 * d * f) + 3 * 2 * 2 * n * d * (t + 1) / 2


def work(case):
    c, fam = case, case["family"]
    es = 2 if c.get("dtype") == "bf16" else 4
    if fam == "chain":
        return {"bytes": 8.0 * c["n"], "flops": float(c["length"] * c["n"])}
    if fam == "ffn":
        n, d, f = c["tokens"], c["d"], c["ff"]
        # in: a, dy, both weights, biases, residual; out: h, y, da, both weight gradients, bias gradient
        return {"bytes": float(es * (2 * n * d + 2 * d * f + n * f + n * d) + 4 * (2 * n * d + 2 * d * f + 2 * f + d)),
                "flops": 12.0 * n * d * f}
    if fam == "attention":
        b, tq, tk, h, hd = c["batch"], c["tq"], c["tk"], c["heads"], c["hd"]
        d, pairs = h * hd, tq * (tq + 1) / 2 if c["role"] == "causal" else tq * tk
        # two products forward, five backward
        return {"bytes": float(es * d * b * (4 * tq + 4 * tk) + 4 * b * h * tq), "flops": 14.0 * b * h * hd * pairs}
    if fam == "layernorm":
        n, d = c["rows"], c["d"]
        return {"bytes": float(n * d * (4 + es + es + 4 + 4 + (es if es == 2 else 0)) + 8 * n + 20 * d), "flops": 0}
    if fam == "head":
        n, d, v = c["batch"] * c["seq"], c["d"], c["vocab"]
        return {"bytes": float(es * (2 * n * d + d * v + n * v) + 4 * d * v + 8 * n), "flops": 6.0 * n * d * v}
    if fam == "embedding":
        n, t, d, v = c["batch"] * c["seq"], c["seq"], c["d"], c["vocab"]
        return {"bytes": 4.0 * d * (min(n, v) + t + n + n + v + t) + 4 * n, "flops": 0}
    if fam == "stage":
        n, d, f, mb = c["batch"] * c["seq"], c["d"], c["ff"], c["microbatches"]
        p = 4 * d * d + 2 * d * f
        return {"bytes": float(mb * 16 * n * d + 30 * p), "flops": mb * _layer_flops(n, c["seq"], d, f)}
    n, d, f, v = c["batch"] * c["seq"], c["d"], c["ff"], c["vocab"]
    p = c["layers"] * (4 * d * d + 2 * d * f) + 2 * v * d + c["seq"] * d
    return {"bytes": float(12 * p + 4 * n * v), "flops": c["layers"] * _layer_flops(n, c["seq"], d, f) + 6.0 * n * d * v}


def tolerance(case):
    return _TOLERANCE[case["family"]] if case["family"] in ("chain", "embedding") else \
        _TOLERANCE[case["family"], case["dtype"]]


# Four times the largest error against 64 bits seen over the listed and fifty drawn cases ("max": largest element).
# bf16 results carry the rounding of their own storage (1.7e-3) and of the operands stored in between; the fp32 ones
# the order of their sums.
_TOLERANCE = {
    "chain": "exact",                       # sequential fp32 additions
    "embedding": {"rel": 2.5e-7, "max": 2e-6},
    ("ffn", "bf16"): {"rel": 1e-2, "max": 5e-2}, ("ffn", "f32"): {"rel": 3e-6, "max": 2e-5},
    ("attention", "bf16"): {"rel": 1e-2, "max": 0.35}, ("attention", "f32"): {"rel": 2e-6, "max": 2e-5},
    ("layernorm", "bf16"): {"rel": 7e-3, "max": 1.6e-2}, ("layernorm", "f32"): {"rel": 1e-6, "max": 1e-5},
    ("head", "bf16"): {"rel": 1e-2, "max": 4e-2},
    ("stage", "bf16"): {"rel": 2.2e-2, "max": 0.1},
    ("lm", "f32"): {"rel": 5e-6, "max": 6e-5}, ("lm", "bf16"): {"rel": 2.5e-2, "max": 0.45},
}


# ---- the same in 64 bits -----------------------------------------------------------------------------------------

def _gelu(u):
    return 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))


def _norm(x, g, b):
    mu = x.mean(-1, keepdim=True)
    var = ((x - mu) ** 2).mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(var + 1e-5) * g + b


def _attend(q, k, v, heads, batch, causal):
    """q [B*Tq, d], k and v [B*Tk, d] -> o [B*Tq, d], lse [B, H, Tq], one batch element at a time."""
    hd = q.shape[1] // heads
    outs, lses = [], []
    for b in range(batch):
        sl = lambda t: t.view(batch, -1, heads, hd)[b].transpose(0, 1)  # noqa: E731
        qq, kk, vv = sl(q), sl(k), sl(v)
        z = torch.matmul(qq, kk.transpose(1, 2)) / math.sqrt(hd)
        if causal:
            z = z.masked_fill(torch.ones(z.shape[1:], dtype=torch.bool, device=z.device).triu(1), -math.inf)
        lse = torch.logsumexp(z, -1)
        outs.append(torch.matmul(torch.exp(z - lse[..., None]), vv).transpose(0, 1).reshape(-1, heads * hd))
        lses.append(lse)
    return torch.cat(outs), torch.stack(lses)


def _layer(x, p, pre, c):
    d = c["d"]
    a = _norm(x, p[pre + "ln1_g"], p[pre + "ln1_b"])
    qkv = a @ p[pre + "wqkv"] + p[pre + "bqkv"]
    o, _ = _attend(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], c["heads"], c["batch"], True)
    x = x + o @ p[pre + "wo"] + p[pre + "bo"]
    m = _norm(x, p[pre + "ln2_g"], p[pre + "ln2_b"])
    return x + _gelu(m @ p[pre + "w1"] + p[pre + "b1"]) @ p[pre + "w2"] + p[pre + "b2"]


def _double(s):
    return {k: v.double() for k, v in s.items()}


def exact(case, seed):
    c, fam = case, case["family"]
    if fam == "chain":
        x = _Draw(seed).normal(c["n"]).cpu().numpy()
        for _ in range(c["length"]):                     # fp32 additions one after the other are the definition
            x = (x + np.float32(1.0)).astype(np.float32)
        return x
    if fam == "ffn":
        s = _double(_ffn_inputs(c, seed))
        u = s["a"] @ s["w1"] + s["b1"]
        u.requires_grad_(True)
        h = _gelu(u)
        (du,) = torch.autograd.grad(h, u, s["dy"] @ s["w2"].T)
        h = h.detach()
        return {"h": h, "y": s["x"] + h @ s["w2"] + s["b2"], "da": du @ s["w1"].T, "dw1": s["a"].T @ du,
                "dw2": h.T @ s["dy"], "db1": du.sum(0)}
    if fam == "attention":
        s, d = _double(_attention_inputs(c, seed)), c["heads"] * c["hd"]
        if c["role"] == "cross":
            ins = [s["q"].requires_grad_(True), s["kv"].requires_grad_(True)]
            q, k, v = ins[0], ins[1][:, :d], ins[1][:, d:]
        else:
            ins = [s["qkv"].requires_grad_(True)]
            q, k, v = ins[0][:, :d], ins[0][:, d:2 * d], ins[0][:, 2 * d:]
        o, lse = _attend(q, k, v, c["heads"], c["batch"], c["role"] == "causal")
        g = torch.autograd.grad(o, ins, s["dout"])
        out = {"o": o.detach(), "lse": lse.detach()}
        out.update({"dq": g[0], "dkv": g[1]} if c["role"] == "cross" else {"dqkv": g[0]})
        return out
    if fam == "layernorm":
        s = _double(_layernorm_inputs(c, seed))
        x, g, b = s["x"].requires_grad_(True), s["g"].requires_grad_(True), s["b"].requires_grad_(True)
        y = _norm(x, g, b)
        dx, dg, db = torch.autograd.grad(y, (x, g, b), s["dy"])
        dx = dx + s["dres"]
        x = x.detach()
        out = {"y": y.detach(), "mean": x.mean(-1), "rstd": 1.0 / torch.sqrt(x.var(-1, unbiased=False) + 1e-5), "dx": dx,
               "dg": dg, "db": db, "dsum": dx.sum(0)}
        if c["dtype"] == "bf16":
            out["dx_lp"] = dx
        return out
    if fam == "head":
        s = _head_inputs(c, seed)
        y, wh, n = s["y"].double(), s["wh"].double(), c["batch"] * c["seq"]
        tgt = s["tokens"][:, 1:].reshape(-1, 1).long()
        z = y @ wh
        lse = torch.logsumexp(z, -1)
        row = lse - z.gather(1, tgt)[:, 0]
        dz = z.sub_(lse[:, None]).exp_()
        dz.scatter_add_(1, tgt, torch.full_like(tgt, -1, dtype=torch.float64))
        dz /= n
        return {"loss": row.mean()[None], "row_loss": row, "z": dz, "dy": dz @ wh.T, "dwh": y.T @ dz}
    if fam == "embedding":
        s = _embedding_inputs(c, seed)
        ids, d = s["tokens"][:, :-1].reshape(-1).long(), c["d"]
        dx = s["dx"].double()
        x = s["wte"].double()[ids] + s["wpe"].double().repeat(c["batch"], 1)
        return {"x": x, "dwte": torch.zeros(c["vocab"], d, dtype=torch.float64, device="cuda").index_add_(0, ids, dx),
                "dwpe": dx.view(c["batch"], c["seq"], d).sum(0)}
    if fam == "stage":
        p, xs, dys = _stage_inputs(c, seed)
        p = {k: v.double().requires_grad_(True) for k, v in p.items()}
        ys, dxs, total = [], [], None
        names = list(p)
        for x, dy in zip(xs, dys):
            x = x.double().requires_grad_(True)
            y = _layer(x, p, "l0.", c)
            g = torch.autograd.grad(y, [x] + [p[k] for k in names], dy.double())
            ys.append(y.detach())
            dxs.append(g[0])
            total = list(g[1:]) if total is None else [a + b for a, b in zip(total, g[1:])]
        grads = dict(zip(names, total))
        return {"y": ys, "dx": dxs, "grads": {k: grads[k] for k in _STAGE_READ}}
    p, tok = _lm_inputs(c, seed)
    p = {k: v.double().requires_grad_(True) for k, v in p.items()}
    ids, tgt = tok[:, :-1].reshape(-1).long(), tok[:, 1:].reshape(-1).long()
    x = p["wte"][ids] + p["wpe"].repeat(c["batch"], 1)
    for i in range(c["layers"]):
        x = _layer(x, p, "l%d." % i, c)
    z = _norm(x, p["lnf_g"], p["lnf_b"]) @ p["wh"]
    loss = torch.nn.functional.cross_entropy(z, tgt)
    names = list(p)
    g = torch.autograd.grad(loss, [z] + [p[k] for k in names])
    return {"loss": loss.detach()[None], "dlogits": g[0].reshape(-1),
            "grads": {k: t.reshape(-1) for k, t in zip(names, g[1:])}}
