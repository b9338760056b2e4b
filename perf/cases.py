"""Performance cases of the library: the calls a program makes of it, with the
sizes it makes them with, the inputs they meet and what each pass cannot do
without.

Decoder calls run on the shapes the framework is configured for: a
Llama-3-8B-shaped and a Qwen3-8B-shaped bf16 decoder (full width and vocabulary,
a few of their layers, so that a pass is short and its inputs quick to make) and
the tiny float32 decoder.  Raw-pointer calls (sampling filter, isolated
knapsack, hidden-state cosine) take the sizes of the same workloads.

Weights are N(0, 0.02^2), output projections smaller, norm gains around 1; cache
contents have the scale of a random-init model's keys and values.  Every input
is drawn on the GPU from the case's seed.
"""
from __future__ import annotations

import ctypes as C
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2602_20217_amd import _lib as K
from paper_2602_20217_amd import engine as E

SHAPES = {
    "llama8b": dict(depth=32, d=4096, hq=32, hkv=8, hd=128, ffn=14336, vocab=128256, eps=1e-6,
                    rope_theta=5e5, qk_norm=False, dtype="bf16"),
    "qwen8b": dict(depth=36, d=4096, hq=32, hkv=8, hd=128, ffn=12288, vocab=151936, eps=1e-6,
                   rope_theta=1e6, qk_norm=True, dtype="bf16"),
    "tiny": dict(depth=4, d=256, hq=4, hkv=2, hd=64, ffn=1024, vocab=1024, eps=1e-6,
                 rope_theta=1e4, qk_norm=False, dtype="f32"),
}
# latency model of a selection (ms): t_MLP = C1, t_Attn(n) = C2 n + C3, the fit
# over context lengths that the benchmark's sweep gives on an MI355X
C1, C2, C3 = 0.0582, 0.69e-6, 0.0278
M_ROUNDS = 5


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: one verify round of the float32 decoder (gamma 4)
        dict(name="tiny_verify", kind="step", model="tiny", layers=4, ctx=131, rows=5),
        # one autoregressive / draft step at 8K context (one row, every sublayer)
        dict(name="llama_decode_8k", kind="step", model="llama8b", layers=4, ctx=8189, rows=1),
        # the verify pass of a round of the 8K workload (gamma 4)
        dict(name="llama_verify_8k", kind="step", model="llama8b", layers=4, ctx=8187, rows=5),
        # the verify pass of the 32K workload (gamma 6, q/k norms, long cache)
        dict(name="qwen_verify_32k", kind="step", model="qwen8b", layers=4, ctx=32765, rows=7),
        # the prompt of the 8K workload
        dict(name="llama_prefill_8k", kind="prefill", model="llama8b", layers=2, n=8192, chunk=512),
        # a short prompt of ragged length, at DeviceModel's default chunk
        dict(name="qwen_prefill_1237", kind="prefill", model="qwen8b", layers=2, n=1237, chunk=256),
        # one mask selection of the 8K workload (25 history rows)
        dict(name="llama_select_8k", kind="select", model="llama8b", layers=16, ctx=8192, gamma_max=4),
        # the candidate rows of one DP stage of the 32K workload's selection
        # (37 budgets x 35 history rows): attention, then MLP
        dict(name="qwen_candidates_32k", kind="candidates", model="qwen8b", layers=1, ctx=32768,
             rows=1295, history=35),
        # logits of a few rows: final norm, LM head, argmax
        dict(name="llama_head_5", kind="head", model="llama8b", rows=5),
        # the T / top-k / top-p filter and draw of the paper's sampling setting
        dict(name="sample_filter_5", kind="sample", rows=5, vocab=128256, top_k=50, top_p=0.95,
             temperature=0.7),
        # the isolated knapsack batch: DP and stage 2 of 1024 instances
        dict(name="knapsack_1024", kind="knapsack", B=1024, items=72, bins=4096, D=10),
        # hidden-state cosines of one DP stage's candidates (49 budgets x 25 rows)
        dict(name="cos_49x25", kind="cos", groups=49, rows=25, d=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "prefill", "prefill", "select", "candidates",
                       "candidates", "head", "sample", "knapsack", "cos"])
    big = rng.choice(["llama8b", "qwen8b"])
    if kind == "step":
        if rng.random() < 0.2:
            return dict(kind=kind, model="tiny", layers=4, ctx=_log(rng, 1, 900),
                        rows=rng.randint(1, 16))
        return dict(kind=kind, model=big, layers=rng.randint(1, 4), ctx=_log(rng, 100, 65536),
                    rows=rng.choice([1, 1, rng.randint(2, 16)]))
    if kind == "prefill":
        if rng.random() < 0.2:
            return dict(kind=kind, model="tiny", layers=4, n=_log(rng, 1, 1000), chunk=64)
        return dict(kind=kind, model=big, layers=rng.randint(1, 2), n=_log(rng, 16, 8000),
                    chunk=rng.choice([64, 256, 256, 512, 512, 1024, 4096]))
    if kind == "select":
        return dict(kind=kind, model=big, layers=rng.randint(2, 14), ctx=_log(rng, 256, 8192),
                    gamma_max=rng.randint(2, 5))
    if kind == "candidates":
        r = rng.randint(10, 45)
        return dict(kind=kind, model=big, layers=1, ctx=_log(rng, 512, 32768),
                    rows=max(17, r * rng.randint(1, 28)), history=r)
    if kind == "head":
        return dict(kind=kind, model=big, rows=_log(rng, 1, 512))
    if kind == "sample":
        return dict(kind=kind, rows=_log(rng, 1, 16), vocab=16 * _log(rng, 64, 9500),
                    top_k=_log(rng, 1, 60), top_p=round(rng.uniform(0.5, 1.0), 3),
                    temperature=round(rng.uniform(0.3, 1.3), 3))
    if kind == "knapsack":
        return dict(kind=kind, B=_log(rng, 1, 1024), items=rng.randint(8, 72),
                    bins=_log(rng, 64, 4096), D=rng.randint(1, 12))
    return dict(kind=kind, groups=_log(rng, 1, 64), rows=rng.randint(1, 45),
                d=rng.choice([256, 1024, 4096, 4096, rng.randint(100, 4096)]))


# ------------------------------------------------------------------- inputs
def _cfg(case):
    s = dict(SHAPES[case["model"]])
    return SimpleNamespace(L=case.get("layers", 1), **s)


def _rng(seed, part):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1009 + part)


def _wdtype(cfg):
    return torch.bfloat16 if cfg.dtype == "bf16" else torch.float32


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _embeddings(cfg, seed):
    g, dt = _rng(seed, 1), _wdtype(cfg)
    return (_normal(g, (cfg.vocab, cfg.d), 0.02, dt), _normal(g, (cfg.vocab, cfg.d), 0.02, dt))


def _layer(cfg, case, seed, l):
    """Row-major weights and gains of one layer.  The attention's output
    projection is not scaled down with depth, so that its update counts beside
    the MLP's at long contexts too; in a selection the layers' output
    projections differ in scale, as those of a trained decoder do."""
    g, dt = _rng(seed, 100 + l), _wdtype(cfg)
    q, kv, d, f = cfg.hq * cfg.hd, cfg.hkv * cfg.hd, cfg.d, cfg.ffn
    out = 0.02 / math.sqrt(2 * cfg.depth)
    so = sm = 1.0
    if case["kind"] == "select":
        r = np.random.default_rng([int(seed), l])
        so, sm = (float(x) for x in np.exp(r.uniform(math.log(0.3), math.log(3.0), 2)))
    w = {"wq": _normal(g, (q, d), 0.02, dt), "wk": _normal(g, (kv, d), 0.02, dt),
         "wv": _normal(g, (kv, d), 0.02, dt), "wo": _normal(g, (d, q), 0.02 * so, dt),
         "w_gate": _normal(g, (f, d), 0.02, dt), "w_up": _normal(g, (f, d), 0.02, dt),
         "w_down": _normal(g, (d, f), out * sm, dt)}
    for name, n in (("attn_norm", d), ("mlp_norm", d), ("q_norm", cfg.hd), ("k_norm", cfg.hd)):
        w[name] = torch.rand(n, generator=g, device="cuda") + 0.5
    return w


def _cache(cfg, seed, l, n):
    """Keys and values of one layer at positions 0..n-1, [hkv, n, hd]."""
    g = _rng(seed, 10000 + l)
    return tuple(_normal(g, (cfg.hkv, n, cfg.hd), 1.28, _wdtype(cfg)) for _ in range(2))


def _tokens(cfg, seed, n):
    t = torch.randint(0, cfg.vocab, (n,), generator=_rng(seed, 20000), device="cuda")
    return t.cpu().numpy().astype(np.int32)


def _rows(cfg, seed, n):
    """Residual rows at the scale of the token embeddings."""
    return _normal(_rng(seed, 30000), (n, cfg.d), 0.02, torch.float32)


class _Decoder(E.DeviceModel):
    """A DeviceModel whose weights arrive as row-major device tensors."""

    def load(self, weights, layer):
        c, dt, st = self.cfg, self.desc.dtype, torch.cuda.current_stream().cuda_stream
        p = lambda t: t.data_ptr()
        qkv = torch.cat([weights["wq"], weights["wk"], weights["wv"]])
        K.ks_pack_qkv(p(qkv), p(self.w["wqkv"][layer]), c.hq, c.hkv, c.hd, c.d, dt, st)
        for k in ("wo", "w_down"):
            K.ks_pack_matrix(p(weights[k]), p(self.w[k][layer]), *weights[k].shape, dt, st)
        K.ks_pack_gate_up(p(weights["w_gate"]), p(weights["w_up"]), p(self.w["w_gate_up"][layer]),
                          c.ffn, c.d, dt, st)
        for k in ("attn_norm", "mlp_norm", "q_norm", "k_norm"):
            self.gains[k][layer].copy_(weights[k])
        self._done.update((k, layer) for k in E._PER_LAYER)

    def load_embeddings(self, embed, head):
        self.w["embed"].view(embed.dtype).copy_(embed)
        K.ks_pack_matrix(head.data_ptr(), self.w["lm_head"].data_ptr(), *head.shape,
                         self.desc.dtype, torch.cuda.current_stream().cuda_stream)
        self._done.update((("embed", -1), ("lm_head", -1)))


def _decoder(case, seed, n_max, gamma_max=8, chunk=512):
    cfg = _cfg(case)
    dm = _Decoder(cfg, n_max=n_max, gamma_max=gamma_max, m_rounds=M_ROUNDS, cap_max=256,
                  prefill_chunk=chunk)
    dm.load_embeddings(*_embeddings(cfg, seed))
    for l in range(cfg.L):
        dm.load(_layer(cfg, case, seed, l), l)
    return cfg, dm.finalize()


def _knapsack_inputs(case, seed):
    """Latencies of attention (a + b ctx) and MLP sublayers in turn at contexts
    log-uniform in [1K, 128K], similarity scores in [0.9, 1]."""
    B, n = case["B"], case["items"]
    g = np.random.default_rng([int(seed), 7])
    ctx = np.exp(g.uniform(math.log(1024), math.log(131072), B))[:, None]
    jit = g.uniform(0.9, 1.1, (3, B, n))
    t = np.where(np.arange(n) % 2 == 0, 10.49e-6 * jit[0] + 0.512e-9 * jit[1] * ctx,
                 44.04e-6 * jit[2])
    return t, g.uniform(0.9, 1.0, (B, n))


def _history(case):
    """Rows that a prefill leaves as the first history block."""
    return min(case["ctx"], M_ROUNDS * (case["gamma_max"] + 1))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        ctx, rows = case["ctx"], case["rows"]
        cfg, dm = _decoder(case, seed, ctx + rows + 64, gamma_max=max(8, rows - 1))
        for l in range(cfg.L):
            for dst, src in zip(dm.kv_layer(l), _cache(cfg, seed, l, ctx)):
                dst[:, :ctx].copy_(src)
        return dict(case=case, dm=dm, tokens=_tokens(cfg, seed, rows))
    if kind == "prefill":
        cfg, dm = _decoder(case, seed, case["n"] + 64, chunk=case["chunk"])
        return dict(case=case, dm=dm, tokens=_tokens(cfg, seed, case["n"]))
    if kind == "select":
        cfg, dm = _decoder(case, seed, case["ctx"] + 320, gamma_max=case["gamma_max"])
        dm.prefill(_tokens(cfg, seed, case["ctx"]))
        return dict(case=case, dm=dm, cells=_capacity(case)[3] + 1,
                    params=E.select_params((C1, C2, C3), "paper_min", 0, tau=0.5, D=10))
    if kind == "candidates":
        ctx, rows, r = case["ctx"], case["rows"], case["history"]
        cfg, dm = _decoder(case, seed, ctx + 64)
        for dst, src in zip(dm.kv_layer(0), _cache(cfg, seed, 0, ctx)):
            dst[:, :ctx].copy_(src)
        return dict(case=case, dm=dm, x=_rows(cfg, seed, rows),
                    pos=(ctx - r + np.arange(rows) % r).astype(np.int32),
                    mid=torch.empty(rows, cfg.d, device="cuda"),
                    out=torch.empty(rows, cfg.d, device="cuda"))
    if kind == "head":
        cfg, dm = _decoder(dict(case, layers=1), seed, 128)
        return dict(case=case, dm=dm, x=_rows(cfg, seed, case["rows"]))
    if kind == "sample":
        R, V, k = case["rows"], case["vocab"], case["top_k"]
        dev = dict(device="cuda")
        return dict(case=case, logits=_normal(_rng(seed, 1), (R, V), 3.0, torch.float32),
                    spec=K.Sampling(case["temperature"], k, case["top_p"], int(seed) + 1),
                    ws=torch.empty(K.ks_sample_workspace_bytes(R, V, k), dtype=torch.uint8, **dev),
                    ids=torch.zeros(R, K.KS_SAMPLE_KMAX, dtype=torch.int32, **dev),
                    probs=torch.zeros(R, K.KS_SAMPLE_KMAX, **dev),
                    counts=torch.zeros(R, dtype=torch.int32, **dev),
                    top1=torch.zeros(R, **dev), tokens=torch.zeros(R, dtype=torch.int32, **dev))
    if kind == "knapsack":
        t, s = _knapsack_inputs(case, seed)
        w, q = E.knapsack_quantize(t, s, case["bins"])
        return dict(case=case, w=torch.from_numpy(w).cuda(), q=torch.from_numpy(q).cuda(),
                    s=torch.from_numpy(s).cuda())
    X, Y = _cos_inputs(case, seed)
    return dict(case=case, X=X, Y=Y)


def _cos_inputs(case, seed):
    """Candidate states: the target rows plus perturbations of several sizes."""
    g = _rng(seed, 1)
    G, r, d = case["groups"], case["rows"], case["d"]
    Y = torch.randn(r, d, generator=g, device="cuda")
    size = torch.rand(G, 1, 1, generator=g, device="cuda")
    return Y + size * torch.randn(G, r, d, generator=g, device="cuda"), Y


# ---------------------------------------------------------------- the passes
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        # one forward of the full model on the committed token and the drafts:
        # target tokens, and the keys / values stored for those rows
        dm, tok, ctx = state["dm"], state["tokens"], case["ctx"]
        dm.set_context(ctx, int(tok[0]))
        pred, _ = dm.verify(tok)
        new = [t[:, ctx:ctx + len(tok)] for l in range(dm.cfg.L) for t in dm.kv_layer(l)]
        return {"pred": pred, "kv": new}
    if kind == "prefill":
        dm, n = state["dm"], case["n"]
        first = dm.prefill(state["tokens"])
        return {"token": first, "kv": [t[:, :n] for l in range(dm.cfg.L) for t in dm.kv_layer(l)]}
    if kind == "select":
        # the decision record (alpha-hat and TPT follow from n_match and the mask)
        dm = state["dm"]
        sel, rec = dm.select(state["params"], debug_cells=state["cells"])
        mask = np.frombuffer(bytes(sel.exec[:2 * dm.cfg.L]), dtype=np.uint8)
        whole = np.concatenate([rec["bits"].ravel(), rec["reach"].ravel(), mask, rec["n_match"],
                                [sel.C, sel.w_attn, sel.w_mlp, sel.n_rows, sel.n_cells]])
        return {"decisions": whole.astype(np.int64), "sig_e": rec["sig_e"], "sig_s": rec["sig_s"]}
    if kind == "candidates":
        dm = state["dm"]
        dm.sublayer_apply(1, state["x"], state["pos"], mode=1, out=state["mid"])
        dm.sublayer_apply(2, state["mid"], state["pos"], mode=1, out=state["out"])
        return {"attention": state["mid"], "mlp": state["out"]}
    if kind == "head":
        logits, argmax, top1 = state["dm"].head_rows(state["x"])
        return {"logits": logits, "argmax": argmax, "top1": top1}
    if kind == "sample":
        s, p = state, lambda t: t.data_ptr()
        R, V = s["logits"].shape
        K.ks_sample_filter(p(s["logits"]), R, V, V, C.byref(s["spec"]), 100, 2, p(s["ids"]),
                           p(s["probs"]), p(s["counts"]), p(s["top1"]), p(s["tokens"]), p(s["ws"]),
                           s["ws"].numel(), torch.cuda.current_stream().cuda_stream)
        return {"table": [s["ids"], s["counts"], s["tokens"]], "probs": s["probs"],
                "top1": s["top1"]}
    if kind == "knapsack":
        cap = case["bins"]
        best, bits = E.knapsack_batch(state["w"], state["q"], cap, cap // 2)
        js, gs, tpt, skip = E.knapsack_batch_select(best, bits, state["w"], state["s"], cap,
                                                    case["D"])
        return {"best": best, "bits": bits, "j": js, "gamma": gs, "tpt": tpt, "skip": skip}
    return E.hidden_cos(state["X"], state["Y"])


# ------------------------------------------------------------ work and errors
def _params(cfg):
    """Weights of one attention and of one MLP sublayer."""
    qkv = (cfg.hq + 2 * cfg.hkv) * cfg.hd
    return cfg.d * (qkv + cfg.hq * cfg.hd), 3 * cfg.d * cfg.ffn


def _capacity(case):
    """Integer weights, capacity and largest skip budget of a selection."""
    ta, tm = C2 * case["ctx"] + C3, C1
    wa, wm = (max(1, math.floor(t / min(ta, tm) + 0.5)) for t in (ta, tm))
    cap = case["layers"] * (wa + wm)
    return wa, wm, cap, cap // 2


def work(case):
    kind = case["kind"]
    if kind == "sample":
        n = case["rows"] * case["vocab"]
        return {"bytes": 4 * n, "flops": 4 * n}
    if kind == "knapsack":
        B, n, cap = case["B"], case["items"], case["bins"]
        cells = B * n * (cap // 2 + 1)
        # best and the decision bits are written, then read by stage 2; three
        # integer operations per cell update
        return {"bytes": 2 * B * (4 * (cap + 1) + 8 * n * (cap // 64 + 1)) + 16 * B * n,
                "flops": 3 * cells}
    if kind == "cos":
        n = case["rows"] * case["d"]
        return {"bytes": 4 * n * (case["groups"] + 1), "flops": 6 * n * case["groups"]}
    cfg = _cfg(case)
    es = 2 if cfg.dtype == "bf16" else 4
    pa, pm = _params(cfg)
    head, kv = cfg.vocab * cfg.d, 2 * cfg.hkv * cfg.hd  # cache elements of a position
    att = 4 * cfg.hq * cfg.hd  # operations of a (row, key) pair
    L = cfg.L
    if kind == "head":
        R = case["rows"]
        return {"bytes": es * head + 4 * R * (cfg.d + cfg.vocab), "flops": 2 * R * head}
    if kind == "step":
        R, ctx = case["rows"], case["ctx"]
        return {"bytes": es * (L * (pa + pm + (ctx + R) * kv) + head),
                "flops": 2 * R * (L * (pa + pm) + head) + L * R * att * ctx}
    if kind == "prefill":
        n = case["n"]
        return {"bytes": es * (L * (pa + pm + n * kv) + head + n * cfg.d),
                "flops": 2 * n * L * (pa + pm) + 2 * head + L * att * n * (n + 1) // 2}
    if kind == "candidates":
        R, ctx = case["rows"], case["ctx"]
        return {"bytes": es * (pa + pm + ctx * kv) + 12 * R * cfg.d,
                "flops": 2 * R * (pa + pm) + R * att * ctx}
    wa, wm, cap, J = _capacity(case)  # select
    r, ctx = _history(case), case["ctx"]
    flops, budgets = 0, {0}
    for i in range(2 * L):
        M = len(budgets) * r
        flops += 2 * M * (pm if i % 2 else pa) + (0 if i % 2 else M * att * ctx)
        budgets |= {j + (wm if i % 2 else wa) for j in budgets}
        budgets = {j for j in budgets if j <= J}
    flops += 2 * (len(budgets) + 1) * r * head
    return {"bytes": es * (L * (pa + pm + ctx * kv) + head), "flops": flops}


def tolerance(case):
    """About four times what outputs moved by when the same inputs ran with
    other split-K factors and attention splits (or, for the float32 paths, four
    times their distance from the same in 64 bits)."""
    kind = case["kind"]
    if kind == "knapsack":
        return "exact"
    if kind == "cos":
        return {"rel": 5e-7, "max": 2e-6}
    if kind == "sample":
        return {"rel": 1e-6, "max": 1e-5, "differ": 2e-3}
    if case.get("model") == "tiny":
        return {"rel": 4e-6, "max": 4e-5}
    if kind == "step":  # keys and values are stored in bf16
        return {"rel": 4e-3, "max": 3e-2}
    if kind == "prefill":  # single bf16 activations through two layers
        return {"rel": 2e-2, "max": 0.12}
    if kind == "select":  # near ties may fall the other way
        return {"rel": 5e-4, "max": 5e-3, "differ": 0.01}
    if kind == "head":  # up to 16 rows: activations as two bf16 planes
        return ({"rel": 1e-5, "max": 1e-4} if case["rows"] <= 16 else {"rel": 1e-2, "max": 5e-2})
    return {"rel": 2e-2, "max": 0.1}


# ------------------------------------------------------- the same in 64 bits
def _norm64(x, g, eps):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, theta):
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    ang = pos.double()[:, None, None] * inv
    c, s, a, b = ang.cos(), ang.sin(), x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attention64(cfg, w, x, pos, past, own):
    """Attention sublayer of rows x [R, d] at pos [R] over the cached keys and
    values `past`: with own, row t sees cache positions below its own and its
    own key / value; otherwise positions below the first row and the rows up to
    its own.  Cached values are rounded to the cache's type.  Returns the
    residual rows, and the keys and values before that rounding."""
    R, G, dt = x.shape[0], cfg.hq // cfg.hkv, _wdtype(cfg)
    h = _norm64(x, w["attn_norm"], cfg.eps)
    q, k, v = ((h @ w[n].double().T).view(R, -1, cfg.hd) for n in ("wq", "wk", "wv"))
    if cfg.qk_norm:
        q, k = _norm64(q, w["q_norm"], cfg.eps), _norm64(k, w["k_norm"], cfg.eps)
    q, k = _rope64(q, pos, cfg.rope_theta), _rope64(k, pos, cfg.rope_theta)
    ks, vs = k.to(dt).double(), v.to(dt).double()
    scale = 1.0 / math.sqrt(cfg.hd)
    o = torch.empty(R, cfg.hq, cfg.hd, dtype=torch.float64, device=x.device)
    for j in range(cfg.hkv):
        pk, pv = past[0][j].double(), past[1][j].double()
        if not own:
            pk, pv = torch.cat([pk, ks[:, j]]), torch.cat([pv, vs[:, j]])
        seen = torch.arange(pk.shape[0], device=x.device)[None, :] < (pos + (not own))[:, None]
        for h_ in range(j * G, (j + 1) * G):
            s = (q[:, h_] @ pk.T * scale).masked_fill_(~seen, -math.inf)
            if own:
                s = torch.cat([s, (q[:, h_] * ks[:, j]).sum(-1, keepdim=True) * scale], 1)
            p = torch.softmax(s, -1)
            o[:, h_] = p[:, :pk.shape[0]] @ pv
            if own:
                o[:, h_] += p[:, -1:] * vs[:, j]
    return x + o.reshape(R, -1) @ w["wo"].double().T, k, v


def _mlp64(cfg, w, x):
    h = _norm64(x, w["mlp_norm"], cfg.eps)
    a = torch.nn.functional.silu(h @ w["w_gate"].double().T) * (h @ w["w_up"].double().T)
    return x + a @ w["w_down"].double().T


def _head64(cfg, x, head):
    return _norm64(x, torch.ones(cfg.d, device=x.device), cfg.eps) @ head.double().T


def _model64(cfg, case, seed, tokens, past_len):
    """All layers on the tokens' rows behind past_len cached positions: the last
    rows, and every layer's new keys and values [hkv, R, hd]."""
    embed, head = _embeddings(cfg, seed)
    x = embed[torch.from_numpy(tokens).long().cuda()].double()
    pos = torch.arange(len(tokens), device="cuda") + past_len
    kv = []
    for l in range(cfg.L):
        w = _layer(cfg, case, seed, l)
        x, k, v = _attention64(cfg, w, x, pos, _cache(cfg, seed, l, past_len), False)
        kv += [k.transpose(0, 1).contiguous(), v.transpose(0, 1).contiguous()]
        x = _mlp64(cfg, w, x)
    return x, head, kv


def _knapsack64(case, seed):
    """TPT of the best (budget, gamma) of every instance: the minimum-loss DP
    over budgets with the acceptance product carried along each chosen path."""
    t, s = _knapsack_inputs(case, seed)
    w, q = E.knapsack_quantize(t, s, case["bins"])
    B, n, cap, D = case["B"], case["items"], case["bins"], case["D"]
    J = cap // 2
    w, q, s = (torch.from_numpy(a).cuda() for a in (w, q, s))
    inf = 1 << 40
    best = torch.full((B, J + 1), inf, device="cuda", dtype=torch.int64)
    alpha = torch.zeros(B, J + 1, device="cuda", dtype=torch.float64)
    best[:, 0], alpha[:, 0] = 0, 1.0
    j = torch.arange(J + 1, device="cuda")[None]
    for i in range(n):
        src = j - w[:, i:i + 1].long()
        skip = best.gather(1, src.clamp(min=0)) + q[:, i:i + 1]
        take = (src >= 0) & (skip < best)
        alpha = torch.where(take, alpha.gather(1, src.clamp(min=0)) * s[:, i:i + 1], alpha)
        best = torch.where(take, skip, best)
    W = w.sum(1, keepdim=True).double()
    top = torch.zeros(B, device="cuda", dtype=torch.float64)
    e, p = torch.ones_like(alpha), alpha.clone()
    for g in range(1, D + 1):
        e, p = e + p, p * alpha
        v = torch.where(best < inf, e / (g * (W - j) + W), 0.0)
        top = torch.maximum(top, v.amax(1))
    return top


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        cfg = _cfg(case)
        x, head, kv = _model64(cfg, case, seed, _tokens(cfg, seed, case["rows"]), case["ctx"])
        return {"pred": _head64(cfg, x, head).argmax(-1).to(torch.int32), "kv": kv}
    if kind == "prefill":
        cfg = _cfg(case)
        x, head, kv = _model64(cfg, case, seed, _tokens(cfg, seed, case["n"]), 0)
        return {"token": int(_head64(cfg, x[-1:], head).argmax()), "kv": kv}
    if kind == "candidates":
        cfg = _cfg(case)
        w = _layer(cfg, case, seed, 0)
        ctx, r = case["ctx"], case["history"]
        pos = ctx - r + torch.arange(case["rows"], device="cuda") % r
        x, _, _ = _attention64(cfg, w, _rows(cfg, seed, case["rows"]).double(), pos,
                               _cache(cfg, seed, 0, ctx), True)
        return {"attention": x, "mlp": _mlp64(cfg, w, x)}
    if kind == "head":
        cfg = _cfg(dict(case, layers=1))
        logits = _head64(cfg, _rows(cfg, seed, case["rows"]).double(), _embeddings(cfg, seed)[1])
        return {"logits": logits, "argmax": logits.argmax(-1).to(torch.int32),
                "top1": torch.softmax(logits, -1).amax(-1)}
    if kind == "sample":
        z = _normal(_rng(seed, 1), (case["rows"], case["vocab"]), 3.0, torch.float32).double()
        top = torch.sort(z, descending=True, stable=True)[0][:, :case["top_k"]]
        p = torch.softmax(top / case["temperature"], -1)
        c = p.cumsum(-1)
        p = torch.where(c - p < case["top_p"], p, 0.0)  # the shortest prefix reaching top_p
        probs = torch.zeros(case["rows"], K.KS_SAMPLE_KMAX, dtype=torch.float64, device="cuda")
        probs[:, :p.shape[1]] = p / p.sum(-1, keepdim=True)
        return {"table": None, "probs": probs, "top1": torch.softmax(z, -1).amax(-1)}
    if kind == "knapsack":
        return {"best": None, "bits": None, "j": None, "gamma": None,
                "tpt": _knapsack64(case, seed), "skip": None}
    if kind == "cos":
        X, Y = (t.double() for t in _cos_inputs(case, seed))
        return ((X * Y).sum(-1) / (X.norm(dim=-1) * Y.norm(dim=-1))).mean(-1)
    return None  # a selection: each decision hangs on the ones before it
