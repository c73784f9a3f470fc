"""Timed cases of the TADM reverse-diffusion step on one GPU.

Each case is work that a serving or evaluation program has the library do, called through
the Python binding exactly as such a program calls it: a reverse step with or without an
anchor refresh, an anchor pass, a context prefill, the sampler on given logits, a step of
the entropy-bound sampler and the pretraining objective's forward pass.  The model shapes
are those of the repository's workloads; where a workload has many equal layers a case may
run fewer of them, so that its outputs can be compared (the change of a rounding grows with
every layer it travels through) and its weights are made quickly.
"""
import math

import numpy as np
import torch

import paper_2609_37924_amd as tadm

# vocabulary, widths and kinds of the five workload models
MODELS = {
    "tiny": dict(dtype="f32", vocab=256, d_model=64, n_heads=4, n_kv_heads=4, head_dim=16, d_ffn=256,
                 ffn_kind="gelu", fusion_kind="gated_mlp", fusion_rank=0),
    "small": dict(dtype="bf16", vocab=32768, d_model=768, n_heads=12, n_kv_heads=12, head_dim=64, d_ffn=2048,
                  ffn_kind="swiglu", fusion_kind="gated_mlp", fusion_rank=0),
    "block": dict(dtype="bf16", vocab=128256, d_model=2048, n_heads=16, n_kv_heads=4, head_dim=128, d_ffn=8192,
                  ffn_kind="swiglu", fusion_kind="gated_mlp", fusion_rank=0),
    "1b": dict(dtype="bf16", vocab=50304, d_model=2048, n_heads=16, n_kv_heads=16, head_dim=128, d_ffn=8192,
               ffn_kind="gelu", fusion_kind="gated_mlp", fusion_rank=0),
    "26b": dict(dtype="bf16", vocab=262144, d_model=4608, n_heads=32, n_kv_heads=16, head_dim=128, d_ffn=36864,
                ffn_kind="geglu", fusion_kind="paired", fusion_rank=256),
}
RMS_EPS, LN_EPS, THETA, PAIRED_HEADS = 1e-6, 1e-5, 10000.0, 4


def _case(op, model, batch, prompt, gen, ctx, anchor, denoise, i, T, **more):
    """prompt + gen: the window of a call; ctx: committed context before it; gen * i // T of
    the generated positions of every row are masked."""
    return dict(op=op, model=model, batch=batch, prompt=prompt, gen=gen, ctx=ctx, anchor=anchor, denoise=denoise,
                i=i, T=T, **more)


def listed():
    return [
        # the smallest call: one float32 row, a refresh step with its logits (launches and latency)
        dict(_case("step", "tiny", 1, 8, 24, 0, 2, 1, 13, 16), name="tiny_step"),
        # one user's canvas on the small model at its full depth: refresh step with logits
        dict(_case("step", "small", 1, 128, 256, 0, 12, 2, 41, 64), name="small_step_b1"),
        # three of four steps of a batched generation: the cached anchor, masked-only head
        dict(_case("denoise", "small", 8, 128, 256, 0, 1, 2, 32, 64), name="small_denoise_b8"),
        # a refresh step of the entropy-bound sampler with self-conditioning, full depth
        dict(_case("entropy", "small", 8, 128, 256, 0, 12, 2, 32, 64), name="small_entropy_b8"),
        # forward pass of the pretraining objective on an odd sequence length
        dict(_case("train", "small", 8, 0, 381, 0, 4, 2, 1, 1), name="small_train_b8"),
        # anchor refresh of one block of one user behind a context (weights streamed once)
        dict(_case("anchor", "block", 1, 0, 64, 711, 4, 0, 16, 32), name="block_anchor_b1"),
        # refresh step of block diffusion, 16 users, masked-only head, ragged context
        dict(_case("refresh", "block", 16, 0, 64, 767, 2, 1, 20, 32), name="block_refresh_b16"),
        # prefill of 16 prompts into the per-layer context
        dict(_case("context", "block", 16, 0, 512, 0, 2, 1, 1, 1), name="block_context_b16"),
        # nucleus sampling with remasking on given logits
        dict(_case("sample", "block", 16, 0, 64, 0, 0, 0, 24, 32, top_p=0.9), name="block_nucleus_b16"),
        # the largest batch: anchor layers over 32 canvases of 1024 tokens
        dict(_case("anchor", "1b", 32, 0, 1024, 0, 2, 0, 64, 128), name="1b_anchor_b32"),
        # a cached-anchor step of the same batch with half of its positions masked
        dict(_case("denoise", "1b", 32, 0, 1024, 0, 1, 1, 64, 128), name="1b_denoise_b32"),
        # refresh step of the post-trained 26B-class shape: paired fusion, masked-only head
        dict(_case("refresh", "26b", 4, 0, 256, 1280, 1, 1, 32, 64), name="26b_refresh_b4"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = {k: max(work(c)[k] for c in listed()) for k in ("flops", "bytes")}
    while True:
        kind = rng.randrange(12)
        T = rng.choice([16, 32, 64, 128])
        i = rng.randint(max(1, T // 8), T)
        if kind == 0:
            c = _case("step", "tiny", log(1, 8), rng.randint(0, 40), log(8, 96), 0, 2, 1, i, T)
        elif kind == 1:
            c = _case("step", "small", log(1, 4), rng.randint(0, 160), log(32, 320), 0, 12, 2, i, T)
        elif kind == 2:
            c = _case("denoise", "small", log(1, 32), rng.randint(0, 160), log(32, 320), 0, 1, 2, i, T)
        elif kind == 3:
            c = _case("entropy", "small", log(1, 8), rng.randint(0, 160), log(32, 320), 0, 6, 2, max(2, i), T)
        elif kind == 4:
            c = _case("train", "small", log(1, 16), 0, log(64, 512), 0, 4, 2, 1, 1)
        elif kind == 5:
            c = _case("anchor", "block", log(1, 4), 0, rng.choice([16, 32, 48, 64, 61]), log(64, 960), 4, 0, i, T)
        elif kind == 6:
            c = _case("refresh", "block", log(2, 24), 0, rng.choice([32, 64, 61]), log(64, 960), 2, 1, i, T)
        elif kind == 7:
            c = _case("context", "block", log(1, 16), 0, log(17, 768), 0, 2, 1, 1, 1)
        elif kind == 8:
            c = _case("sample", rng.choice(["small", "block", "1b"]), log(1, 16), rng.randint(0, 24), log(16, 128), 0,
                      0, 0, i, T, top_p=rng.choice([0.0, 0.8, 0.9, 0.95]))
        elif kind == 9:
            c = _case("anchor", "1b", log(1, 32), 0, log(100, 1024), 0, 2, 0, i, T)
        elif kind == 10:
            c = _case("denoise", "1b", log(1, 32), 0, log(100, 1024), 0, 1, 1, i, T)
        else:
            c = _case("refresh", "26b", log(1, 4), 0, rng.choice([64, 128, 256, 251]), log(64, 1280), 1, 1, i, T)
        w = work(c)
        if w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"]:
            return c


# ------------------------------------------------------------------------------ sizes
def _config(case):
    c = dict(MODELS[case["model"]], n_shared=0, n_anchor=case["anchor"], n_denoise=case["denoise"],
             paired_heads=PAIRED_HEADS, rms_eps=RMS_EPS, ln_eps=LN_EPS, rope_theta=THETA)
    if case["op"] == "sample":  # the sampler reads no layer and no weight: the smallest model of that vocabulary
        c.update(d_model=64, n_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64)
    return c


def _specs(c):
    """(name, shape, kind) of every weight in the library's order."""
    d, V, H, Hk, dh, F, r = (c["d_model"], c["vocab"], c["n_heads"], c["n_kv_heads"], c["head_dim"], c["d_ffn"],
                             c["fusion_rank"])
    s = [("embed", (V + 1, d), 0), ("final_norm", (d,), 1), ("w_out", (V, d), 0)]
    if c["fusion_kind"] == "gated_mlp":
        s += [("ln_s_w", (d,), 1), ("ln_s_b", (d,), 2), ("ln_a_w", (d,), 1), ("ln_a_b", (d,), 2),
              ("w1", (4 * d, 2 * d), 0), ("b1", (4 * d,), 2), ("wg", (d, 2 * d), 0), ("bg", (d,), 2),
              ("w2", (d, 4 * d), 0), ("b2", (d,), 2), ("ln_o_w", (d,), 1), ("ln_o_b", (d,), 2)]
    else:
        s += [("w_c", (r, d), 0), ("w_h", (r, d), 0), ("w_q", (r, 2 * r), 0), ("w_k", (r, 2 * r), 0),
              ("w_v", (r, 2 * r), 0), ("w_o", (r, r), 0), ("w_f1", (2 * r, r), 0), ("w_f2", (r, 2 * r), 0),
              ("w_g1", (r, 4 * r), 0), ("w_g2", (1, r), 0), ("b_g", (1,), 3), ("w_up", (d, r), 0)]
    for li in range(c["n_anchor"] + c["n_denoise"]):
        p = "%d." % li
        s += [(p + "attn_norm", (d,), 1), (p + "wq", (H * dh, d), 0), (p + "wk", (Hk * dh, d), 0),
              (p + "wv", (Hk * dh, d), 0), (p + "wo", (d, H * dh), 0), (p + "ffn_norm", (d,), 1)]
        if c["ffn_kind"] != "gelu":
            s.append((p + "w_gate", (F, d), 0))
        s += [(p + "w_up", (F, d), 0), (p + "w_down", (d, F), 0)]
    return s


def work(case):
    """Products of the pass (2 flops per multiply-add) and every weight, input and output once."""
    c = _config(case)
    op, B, L, ctx = case["op"], case["batch"], case["prompt"] + case["gen"], case["ctx"]
    d, V, H, Hk, dh, F, r = (c["d_model"], c["vocab"], c["n_heads"], c["n_kv_heads"], c["head_dim"], c["d_ffn"],
                             c["fusion_rank"])
    es = 2 if c["dtype"] == "bf16" else 4
    N, rows = B * L, B * case["gen"]
    masked = B * (case["gen"] * case["i"] // case["T"])
    if op == "sample":  # about 40 operations a logit: the counter-based generator, logarithms, exponential
        return {"bytes": masked * V * 4 + B * L * 12, "flops": masked * V * 40}
    per_layer = d * (H + 2 * Hk) * dh + H * dh * d + (2 if c["ffn_kind"] == "gelu" else 3) * d * F
    lf = 2 * N * per_layer + 4 * N * (ctx + L) * H * dh
    lb = per_layer * es + 2 * B * ctx * Hk * dh * es
    if r:
        fuse_p = d * r + 6 * r * r + r * r + 4 * r * r + 4 * r * r + d * r
        ff = 2 * N * fuse_p + 4 * N * L * r
    else:
        fuse_p = 10 * d * d + 4 * d * d
        ff = 2 * N * fuse_p
    anchor = (case["anchor"] * lf, case["anchor"] * lb)
    den = (case["denoise"] * lf + ff, case["denoise"] * lb + fuse_p * es)
    embed = N * d * es + N * 4
    if op == "anchor":
        f, b = anchor[0], anchor[1] + embed + N * d * 4
    elif op == "context":
        f, b = anchor[0] + den[0], anchor[1] + den[1] + embed + (case["anchor"] + case["denoise"]) * 2 * N * Hk * dh * es
    elif op == "denoise":
        f, b = den[0] + 2 * masked * V * d, den[1] + embed + N * d * 4 + V * d * es
    elif op == "refresh":
        f, b = anchor[0] + den[0] + 2 * masked * V * d, anchor[1] + den[1] + embed + V * d * es
    elif op == "step":
        f, b = anchor[0] + den[0] + 2 * rows * V * d, anchor[1] + den[1] + embed + V * d * es + rows * V * 4
    elif op == "entropy":  # head and self-conditioning product over every canvas row
        f, b = anchor[0] + den[0] + 4 * rows * V * d, anchor[1] + den[1] + embed + 2 * V * d * es + rows * V * 4
    else:  # train: the head over the masked half of the tokens
        f, b = anchor[0] + den[0] + N * V * d, anchor[1] + den[1] + 2 * embed + V * d * es
    return {"bytes": b, "flops": f}


# ----------------------------------------------------------------------------- inputs
def _generator(seed, device, n):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1000003 + 7919 * n + 101) & 0x7FFFFFFF)
    return g


def _weight(c, index, spec, seed, device):
    _, shape, kind = spec
    g = _generator(seed, device, index + 10)
    t = torch.randn(shape, generator=g, device=device, dtype=torch.float32)
    if kind == 0:  # matrices: the initialisation of the pretrained shapes
        t *= 0.02
    else:          # norm gains about 1, biases about 0, the paired gate's bias about -3
        t = 0.1 * t + (0.0, 1.0, 0.0, -3.0)[kind]
    return t.to(torch.bfloat16 if c["dtype"] == "bf16" else torch.float32)


def _tokens(case, c, seed, device):
    """(context, window, earlier window) token tensors: int32, the mask id is the vocabulary size.
    The earlier window is the one the cached anchor was computed from, with more masked."""
    B, P, M0, V = case["batch"], case["prompt"], case["gen"], c["vocab"]
    g = _generator(seed, "cpu", 1)
    ctx = torch.randint(0, V, (B, case["ctx"]), generator=g, dtype=torch.int32)
    win = torch.randint(0, V, (B, P + M0), generator=g, dtype=torch.int32)
    old = win.clone()
    n, n_old = M0 * case["i"] // case["T"], M0 * min(case["T"], case["i"] + 2) // case["T"]
    if case["op"] not in ("entropy", "train", "context"):
        for b in range(B):
            p = torch.randperm(M0, generator=g) + P
            win[b, p[:n]] = V
            old[b, p[:n_old]] = V
    return ctx.to(device), win.to(device), old.to(device)


class _State:
    """A program's model, context and anchor cache, given back with the object."""

    def __init__(self):
        self.m = self.ctx = self.cache = None

    def __del__(self):
        if self.cache is not None:
            tadm.tadm_cache_destroy(self.cache)
        if self.ctx is not None:
            tadm.tadm_context_destroy(self.ctx)
        if self.m is not None:
            tadm.tadm_model_destroy(self.m)


def _entropy_eta(case, c):
    """A bound that accepts about half of the canvas at the flat distributions of seeded weights."""
    return 0.5 * case["gen"] * math.log(c["vocab"])


def prepare(case, seed):
    dev = torch.device("cuda")
    c = _config(case)
    s = _State()
    B, P, M0, V, d = case["batch"], case["prompt"], case["gen"], c["vocab"], c["d_model"]
    L = P + M0
    s.case, s.B, s.L, s.P = case, B, L, P
    s.m = tadm.tadm_model_create(tadm.make_config(c, B, case["ctx"] + L))
    for k, spec in enumerate(_specs(c)):
        tadm.tadm_model_load_weight(s.m, k, _weight(c, k, spec, seed, dev))
    tadm.tadm_set_stream(s.m, torch.cuda.current_stream().cuda_stream)
    ctx, s.win, old = _tokens(case, c, seed, dev)
    i, T, op = case["i"], case["T"], case["op"]
    s.next = torch.empty(B, L, dtype=torch.int32, device=dev)
    s.choice = torch.empty(B, M0, dtype=torch.int32, device=dev)
    s.conf = torch.empty(B, M0, dtype=torch.float32, device=dev)
    n = tadm.tadm_unmask_count(M0, i, T)
    if op == "sample":
        s.logits = torch.randn(B, M0, V, generator=_generator(seed, dev, 2), device=dev) * 2.0
        s.args = tadm.step_args(i, T, n, T - i, seed, 1.0, remask=tadm.tadm_remask_probs(i, T, 0.04),
                                top_p=case["top_p"])
        return s
    if case["ctx"] or op == "context":
        s.ctx = tadm.tadm_context_create(s.m, B, case["ctx"] + L)
        if case["ctx"]:
            tadm.tadm_context_append(s.m, s.ctx, ctx, B, case["ctx"])
    if op == "context":
        cap = tadm.tadm_context_capacity(s.ctx)
        shape = (B, c["n_kv_heads"], cap, c["head_dim"])
        s.kv = [(torch.empty(shape, dtype=torch.bfloat16, device=dev), torch.empty(
            (B, c["n_kv_heads"], c["head_dim"], cap), dtype=torch.bfloat16, device=dev))
            for _ in range(case["anchor"] + case["denoise"])]
        return s
    if op == "train":
        t, ts, _, _, _ = tadm.tadm_stale_times(B, seed, 0, 1e-3)
        s.t, s.ts = torch.from_numpy(t).to(dev), torch.from_numpy(ts).to(dev)
        s.loss, s.n = torch.empty(B, device=dev), torch.empty(B, dtype=torch.int32, device=dev)
        s.zt, s.zs, s.seed = torch.empty_like(s.win), torch.empty_like(s.win), seed
        return s
    s.cache = tadm.tadm_cache_create(s.m, B, L)
    s.h = torch.empty(B, L, d, device=dev) if op == "anchor" else None
    if op == "denoise":  # the anchor of an earlier step
        tadm.tadm_anchor_forward(s.m, s.ctx, old, B, L, min(T, i + 2), T, s.cache)
    s.logits = torch.empty(B, M0, V, device=dev) if op in ("step", "entropy") else None
    if op == "entropy":
        s.sc_in = torch.randn(B, M0, d, generator=_generator(seed, dev, 3), device=dev) * 0.01
        s.sc_out = torch.empty_like(s.sc_in)
        s.args = tadm.step_args(i, T, 0, T - i, seed, tadm.tadm_entropy_inv_temp(i, T, 0.8, 0.4),
                                entropy_eta=_entropy_eta(case, c), sc_in=s.sc_in, sc_out=s.sc_out)
    else:
        s.args = tadm.step_args(i, T, n, T - i, seed, 1.0)
    return s


def run(s):
    case, op, B, L, P = s.case, s.case["op"], s.B, s.L, s.P
    i, T = case["i"], case["T"]
    if op == "sample":
        tadm.tadm_sample(s.m, s.logits, s.win, B, L, P, 0, s.args, s.next, s.choice, s.conf)
        return {"next": s.next, "choice": s.choice, "conf": s.conf}
    if op == "context":
        tadm.tadm_context_reset(s.ctx)
        tadm.tadm_context_append(s.m, s.ctx, s.win, B, L)
        for li, (k, vt) in enumerate(s.kv):
            tadm.tadm_context_read(s.ctx, li, k, vt)
        return [{"k": k[:, :, :L], "vt": vt[:, :, :, :L]} for k, vt in s.kv]
    if op == "train":
        tadm.tadm_train_loss(s.m, s.win, B, L, s.t, s.ts, 1e-3, s.seed, 0, s.loss, s.n, s.zt, s.zs)
        return {"loss": s.loss, "masked": s.n, "zt": s.zt, "zs": s.zs}
    if op == "anchor":
        tadm.tadm_anchor_forward(s.m, s.ctx, s.win, B, L, i, T, s.cache)
        tadm.tadm_cache_read(s.cache, tadm.CACHE_H, s.h)
        return {"h": s.h}
    if op == "entropy":
        tadm.tadm_anchor_forward_sc(s.m, s.ctx, s.win, B, L, i, T, s.sc_in, P, s.cache)
        tadm.tadm_denoise_step(s.m, s.ctx, s.win, B, L, P, s.cache, s.args, s.logits, s.next)
        return {"logits": s.logits, "next": s.next, "sc": s.sc_out}
    if op != "denoise":
        tadm.tadm_anchor_forward(s.m, s.ctx, s.win, B, L, i, T, s.cache)
    tadm.tadm_denoise_step(s.m, s.ctx, s.win, B, L, P, s.cache, s.args, s.logits, s.next)
    if op == "step":
        return {"logits": s.logits, "next": s.next}
    tadm.tadm_debug_read(s.m, tadm.TAP_CHOICE, s.choice)
    tadm.tadm_debug_read(s.m, tadm.TAP_CONF, s.conf)
    return {"next": s.next, "choice": s.choice, "conf": s.conf}


def tolerance(case):
    if case["op"] == "sample":  # decisions on given logits: integer sums and rounded float32, any order
        return "exact"
    if case["model"] == "tiny":  # float32 sums
        return {"rel": 2e-6, "differ": 0.01}
    if case["op"] in ("denoise", "refresh"):
        # a log-probability moves with its logit's rounding; where two tokens nearly tie, the
        # other one is drawn and the log-probability of that position changes whole
        return {"rel": 0.03, "max": 0.9, "differ": 0.01}
    if case["op"] == "train":  # sums of many positions' log-probabilities
        return {"rel": 1e-4}
    return {"rel": 0.02, "max": 0.3, "differ": 0.01}


# -------------------------------------------------------------------- 64-bit reference
class _Ref:
    """The networks in float64 on the stored weights, one batch row at a time."""

    def __init__(self, case, seed):
        self.case, self.seed, self.dev = case, seed, torch.device("cuda")
        self.c = _config(case)
        self.specs = {s[0]: (k, s) for k, s in enumerate(_specs(self.c))}
        self.kept = {}

    def w(self, name):
        if name not in self.kept:
            k, s = self.specs[name]
            self.kept[name] = _weight(self.c, k, s, self.seed, self.dev).double()
        return self.kept[name]

    def rms(self, x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + RMS_EPS) * g

    def ln(self, x, w, b):
        mu = x.mean(-1, keepdim=True)
        return (x - mu) / torch.sqrt(((x - mu) ** 2).mean(-1, keepdim=True) + LN_EPS) * w + b

    def gelu(self, x):
        return 0.5 * x * (1 + torch.erf(x / math.sqrt(2.0)))

    def rope(self, x, pos):
        half = x.shape[-1] // 2
        f = THETA ** (-torch.arange(half, dtype=torch.float64, device=self.dev) * 2.0 / x.shape[-1])
        a = pos.double()[:, None] * f[None]
        co, si = torch.cos(a)[:, None], torch.sin(a)[:, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * co - b * si, b * co + a * si], -1)

    def attend(self, q, k, v):
        G = q.shape[1] // k.shape[1]
        out = torch.empty_like(q)
        for h in range(q.shape[1]):
            p = torch.softmax(q[:, h] @ k[:, h // G].T.contiguous() / math.sqrt(q.shape[2]), -1)
            out[:, h] = p @ v[:, h // G]
        return out.reshape(q.shape[0], -1)

    def layer(self, li, x, pos, past, kept):
        c, p, L = self.c, "%d." % li, x.shape[0]
        xn = self.rms(x, self.w(p + "attn_norm"))
        q = self.rope((xn @ self.w(p + "wq").T).reshape(L, c["n_heads"], -1), pos)
        k = self.rope((xn @ self.w(p + "wk").T).reshape(L, c["n_kv_heads"], -1), pos)
        v = (xn @ self.w(p + "wv").T).reshape(L, c["n_kv_heads"], -1)
        if kept is not None:
            kept[li] = (k, v)
        if past is not None:
            k, v = torch.cat([past[li][0], k]), torch.cat([past[li][1], v])
        x = x + self.attend(q, k, v) @ self.w(p + "wo").T
        xn = self.rms(x, self.w(p + "ffn_norm"))
        u = xn @ self.w(p + "w_up").T
        if c["ffn_kind"] == "gelu":
            u = self.gelu(u)
        else:
            g = xn @ self.w(p + "w_gate").T
            u = (g * torch.sigmoid(g) if c["ffn_kind"] == "swiglu" else self.gelu(g)) * u
        return x + u @ self.w(p + "w_down").T

    def embed(self, z):
        return self.w("embed")[z.long()]

    def anchor(self, x, pos, past=None, kept=None):
        for li in range(self.c["n_anchor"]):
            x = self.layer(li, x, pos, past, kept)
        return x

    def mixer(self, Z, U):
        L, r = Z.shape
        J = torch.cat([Z, U], -1)
        q, k, v = ((J @ self.w(n).T).reshape(L, PAIRED_HEADS, -1) for n in ("w_q", "w_k", "w_v"))
        R = Z + self.attend(q, k, v) @ self.w("w_o").T
        f = R @ self.w("w_f1").T
        return R + (f * torch.sigmoid(f)) @ self.w("w_f2").T

    def fuse(self, x, x0, h0):
        if self.c["fusion_kind"] == "gated_mlp":
            u = torch.cat([self.ln(x, self.w("ln_s_w"), self.w("ln_s_b")),
                           self.ln(h0, self.w("ln_a_w"), self.w("ln_a_b"))], -1)
            g = torch.sigmoid(u @ self.w("wg").T + self.w("bg"))
            y = self.gelu(u @ self.w("w1").T + self.w("b1")) @ self.w("w2").T + self.w("b2")
            return self.ln(h0 + g * y, self.w("ln_o_w"), self.w("ln_o_b"))
        sc = torch.sqrt((x0 * x0).mean(-1, keepdim=True) + RMS_EPS)
        sh = torch.sqrt((h0 * h0).mean(-1, keepdim=True) + RMS_EPS)
        Z, Z0, U = (x / sc) @ self.w("w_c").T, (x0 / sc) @ self.w("w_c").T, (h0 / sh) @ self.w("w_h").T
        M = self.mixer(Z, U) - self.mixer(Z0, U)
        f = torch.cat([U, Z0, Z - Z0, M], -1) @ self.w("w_g1").T
        g = torch.sigmoid((f * torch.sigmoid(f)) @ self.w("w_g2").T + self.w("b_g"))
        return h0 + g * sh * (M @ self.w("w_up").T)

    def denoise(self, x, pos, past=None, kept=None):
        for li in range(self.c["n_anchor"], self.c["n_anchor"] + self.c["n_denoise"]):
            x = self.layer(li, x, pos, past, kept)
        return x

    def fresh(self, z, pos):
        """Keys and values of every layer of a fresh pass over clean tokens."""
        kept = {}
        x = self.embed(z)
        h = self.anchor(x, pos, None, kept)
        self.denoise(self.fuse(x, x, h), pos, None, kept)
        return kept

    def head(self, x):
        return self.rms(x, self.w("final_norm")) @ self.w("w_out").T


def _philox(c0, c1, c2, c3, seed):
    """Words of Philox4x32-10 (Salmon et al., SC'11) as int64 tensors holding 32 bits."""
    m = 0xFFFFFFFF
    c = [c0, c1, c2, c3]
    k0, k1 = seed & m, (seed >> 32) & m
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # 64-bit products, wrapped; their halves are exact
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
    return c


def _uniform(w):
    return ((w >> 9) * 2 + 1).double() * 2.0 ** -24


def _draw_tokens(logits, pos, row, step, seed, top_p=0.0):
    """(token, log-probability) of Gumbel-max sampling from rows of float64 logits."""
    V, dev = logits.shape[1], logits.device
    tok = torch.empty(len(pos), dtype=torch.int64, device=dev)
    conf = torch.empty(len(pos), dtype=torch.float64, device=dev)
    q = torch.arange((V + 3) // 4, device=dev)[None]
    for a in range(0, len(pos), 64):
        l = logits[a:a + 64]
        z = torch.zeros_like(q)
        w = _philox(q + 0 * pos[a:a + 64, None], z + pos[a:a + 64, None], z + row, z + step, seed)
        u = _uniform(torch.stack(w, -1).reshape(len(l), -1)[:, :V])
        score = l - torch.log(-torch.log(u))
        p = torch.log_softmax(l, -1)
        if top_p:
            s, order = torch.sort(p, dim=-1, descending=True)
            out = torch.cumsum(s.exp(), -1) - s.exp() >= float(np.float32(top_p))
            score = score.masked_fill(torch.zeros_like(out).scatter(1, order, out), -math.inf)
        tok[a:a + 64] = score.argmax(-1)
        conf[a:a + 64] = p.gather(1, tok[a:a + 64, None])[:, 0]
    return tok, conf


def exact(case, seed):
    with torch.no_grad():
        return _exact(case, seed)


def _exact(case, seed):
    r = _Ref(case, seed)
    c, dev, op = r.c, r.dev, case["op"]
    B, P, M0, V = case["batch"], case["prompt"], case["gen"], c["vocab"]
    L, i, T = P + M0, case["i"], case["T"]
    ctx, win, old = _tokens(case, c, seed, dev)
    if op == "sample":
        lg = torch.randn(B, M0, V, generator=_generator(seed, dev, 2), device=dev) * 2.0
    rows = []
    if op == "train":
        t, ts, _, _, _ = _stale_times(B, seed)
    if op == "entropy":
        sc_in = torch.randn(B, M0, c["d_model"], generator=_generator(seed, dev, 3), device=dev) * 0.01
        inv = 1.0 / (float(np.float32(0.4)) + (float(np.float32(0.8)) - float(np.float32(0.4))) * i / T)
    pos = torch.arange(case["ctx"], case["ctx"] + L, device=dev)
    for b in range(B):
        if op == "sample":
            conf = torch.full((M0,), -math.inf, dtype=torch.float64, device=dev)
            at = (win[b, P:] == V).nonzero()[:, 0]
            conf[at] = _draw_tokens(lg[b, at].double(), P + at, b, T - i, seed, case["top_p"])[1]
            rows.append(conf)
            continue
        past = r.fresh(ctx[b], torch.arange(case["ctx"], device=dev)) if case["ctx"] else None
        if op == "context":
            kv = r.fresh(win[b], pos)
            rows.append([(kv[li][0].transpose(0, 1), kv[li][1].permute(1, 2, 0)) for li in sorted(kv)])
            continue
        if op == "train":
            u = _uniform(_philox(torch.full((L,), 0x80000003, device=dev), torch.arange(L, device=dev),
                                 torch.full((L,), b, device=dev), torch.zeros(L, dtype=torch.int64, device=dev),
                                 seed)[0])
            zt, zs = win[b].clone(), win[b].clone()
            zt[u < _threshold(t[b])] = V
            zs[u < _threshold(ts[b])] = V
            x0 = r.embed(zs)
            x = r.denoise(r.fuse(r.embed(zt), x0, r.anchor(x0, pos)), pos)
            at = (zt == V).nonzero()[:, 0]
            p = torch.log_softmax(r.head(x[at]), -1).gather(1, win[b, at].long()[:, None])
            rows.append(-p.sum() / float(t[b]))
            continue
        x = r.embed(win[b])
        if op == "entropy":
            x[P:] += sc_in[b].double()
        if op == "anchor":
            rows.append(r.anchor(x, pos, past))
            continue
        x0 = r.embed(old[b]) if op == "denoise" else x
        x = r.denoise(r.fuse(x, x0, r.anchor(x0, pos, past)), pos, past)[P:]
        if op == "step":
            rows.append(r.head(x))
        elif op == "entropy":
            lg = r.head(x)
            rows.append((lg, torch.softmax(lg * inv, -1) @ r.w("embed")[:V]))
        else:
            conf = torch.full((M0,), -math.inf, dtype=torch.float64, device=dev)
            at = (win[b, P:] == V).nonzero()[:, 0]
            for a in range(0, len(at), 256):
                k = at[a:a + 256]
                conf[k] = _draw_tokens(r.head(x[k]), case["ctx"] + P + k, b, T - i, seed)[1]
            rows.append(conf)
    if op == "context":
        return [{"k": torch.stack([x[li][0] for x in rows]), "vt": torch.stack([x[li][1] for x in rows])}
                for li in range(case["anchor"] + case["denoise"])]
    if op == "train":
        return {"loss": torch.stack(rows), "masked": None, "zt": None, "zs": None}
    if op == "anchor":
        return {"h": torch.stack(rows)}
    if op == "step":
        return {"logits": torch.stack(rows), "next": None}
    if op == "entropy":
        return {"logits": torch.stack([x[0] for x in rows]), "next": None, "sc": torch.stack([x[1] for x in rows])}
    return {"next": None, "choice": None, "conf": torch.stack(rows)}


def _threshold(t):
    """Probability of a masked position at time t: (1 - eps) t of the log-linear schedule."""
    return float(np.float32((1.0 - float(np.float32(1e-3))) * float(t)))


def _stale_times(B, seed):
    """The binding's own draw of training times: an input of the pass, not a result."""
    return tadm.tadm_stale_times(B, seed, 0, 1e-3)
