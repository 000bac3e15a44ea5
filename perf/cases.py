"""Timed workloads of the library: what its users call, at the sizes they call it.

A case is a dict of plain values; `prepare` makes what a program holds before the call
(states, weights, caches, workspace), `run` is one pass through the public entry points
and `exact` restates the same computation in plain float64 torch. The model shapes are the
repository's own (tests/synth.py, bench.py): the paper's 16-layer model (6 query / 3 KV
heads of 96, every second layer routed), its 4-layer prefill-timing model, a 12-layer and a
24-layer model with heads of 64. Inputs are seeded stand-ins with the distributions of
tests/synth.py; `out_std` is the scale of the stand-in block's output projection.

Kinds:
  step    wm.layer_step: pool, queries and attention of the new tokens in one call
          (T_new = 1..4: decode; larger: a prompt, a chunk of one, or packed documents)
  layers  the depth-sequential decoder's calls for one new token per sequence:
          wm.layer_attend for every layer, then wm.pool
  pool    wm.pool alone (refreshing cache rows from finished states)
  passes  wm.prefill_passes: the fixed-point prefill over g strided groups
  grad    wm.layer_step_backward: the gradients of one full-sequence step
  train   wm.prefill_passes_backward: the training passes with truncated backpropagation
"""
import math

import torch
from torch.utils.checkpoint import checkpoint

import paper_2608_18486_amd as wm

PAPER = dict(L=16, D=512, Hq=6, Hkv=3, d=96, p=2)
FOUR = dict(L=4, D=512, Hq=6, Hkv=3, d=96, p=1)
MID = dict(L=12, D=768, Hq=12, Hkv=12, d=64, p=1)
WIDE = dict(L=24, D=1024, Hq=16, Hkv=16, d=64, p=1)
MODELS = {"paper": PAPER, "four": FOUR, "mid": MID, "wide": WIDE}
CHANNELS = {"paper": (1, 2, 4, 8, 12, 16), "four": (1, 2, 4), "mid": (6, 12), "wide": (6, 12)}

EPS, THETA = 1e-6, 1e6


def _case(kind, model, k, B, T, name=None, **more):
    c = dict(kind=kind, k=k, B=B, T=T, ctx=0, ragged=False, doc_mean=0, dtype="bf16",
             softmax=False, inclusive=False, router=0, groups=1, passes=0, n_grad=0,
             out_std=0.02)
    c.update(MODELS[model])
    c.update(more)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # One user's chat: the next token, layer by layer, over a short context.
        _case("layers", "paper", 8, 1, 1, "decode_b1_ctx700", ctx=709),
        # A batch of long conversations decoding one token each: the cache stream.
        _case("step", "wide", 12, 16, 1, "decode_b16_ctx8k", ctx=8191, ragged=True),
        # Verifying four drafted tokens per sequence of a middling batch.
        _case("step", "paper", 8, 8, 4, "verify4_b8_ctx4k", ctx=4001, ragged=True),
        # A chunk of a long prompt appended to a ragged batch of caches.
        _case("step", "paper", 16, 2, 509, "chunk509_b2_ctx3k", ctx=3001, ragged=True),
        # The full-sequence step of the largest model (the benchmark's headline shape).
        _case("step", "wide", 12, 4, 4096, "step_t4096_l24"),
        # Pretraining rows packed from documents, a batch smaller than the full one.
        _case("step", "paper", 8, 6, 1777, "docs_t1777_b6", doc_mean=512),
        # Single precision at a ragged length.
        _case("step", "mid", 6, 2, 517, "f32_t517_b2", dtype="f32"),
        # Cache rows rebuilt from finished states: no deep-to-shallow feedback, softmax mix.
        _case("pool", "paper", 16, 3, 1023, "pool_t1023_nofb", softmax=True, router=2),
        # The paper's prefill timing: 4 layers, 64 sequences of 2048, 16 groups, 4 passes.
        _case("passes", "four", 4, 64, 2048, "prefill_g16_l4", groups=16, passes=4),
        # Prefill of the 16-layer model for a small serving batch.
        _case("passes", "paper", 8, 4, 2048, "prefill_g8_l16", groups=8, passes=3),
        # The gradients of one full-sequence step.
        _case("grad", "mid", 6, 4, 2048, "grad_t2048_l12"),
        # The paper's training setting on one GPU: 8 groups, 3 passes, 2 with gradients.
        _case("train", "paper", 8, 16, 2048, "train_g8_l16", groups=8, passes=3, n_grad=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "layers", "chunk", "full", "full", "docs", "f32",
                       "pool", "passes", "grad", "train"])
    model = rng.choice(["paper", "paper", "mid", "wide"])
    k = rng.choice(CHANNELS[model])
    opts = dict(softmax=rng.random() < 0.25, inclusive=rng.random() < 0.25)
    if rng.random() < 0.2:
        opts["router"] = 1
    if kind in ("decode", "layers"):
        ctx = _log(rng, 100, 8191)
        B = _log(rng, 1, max(1, min(64, 16 * 8192 // ctx)))
        if kind == "layers":  # a token reads the slots before its own
            opts["inclusive"] = False
            return _case("layers", model, k, min(B, 8), 1, ctx=ctx, ragged=B > 1, **opts)
        T = rng.choice([1, 1, 1, 2, 3, 4])
        return _case("step", model, k, B, T, ctx=ctx, ragged=B > 1, **opts)
    if kind == "chunk":
        T, B = _log(rng, 5, 1024), _log(rng, 1, 4)
        return _case("step", model, k, B, T, ctx=_log(rng, 64, 6000), ragged=B > 1, **opts)
    if kind in ("full", "docs", "pool"):
        T = _log(rng, 100, 4096)
        B = _log(rng, 1, max(1, min(16, 16384 // T)))
        if kind == "docs":
            return _case("step", model, k, B, T, doc_mean=rng.choice([64, 256, 512]), **opts)
        return _case("pool" if kind == "pool" else "step", model, k, B, T, **opts)
    if kind == "f32":
        return _case("step", "mid", rng.choice(CHANNELS["mid"]), _log(rng, 1, 4),
                     rng.choice([1, _log(rng, 5, 700)]), ctx=rng.choice([0, _log(rng, 50, 500)]),
                     dtype="f32", **opts)
    opts.pop("inclusive")
    if kind == "grad":
        T = _log(rng, 100, 2048)
        return _case("grad", model, k, _log(rng, 1, max(1, 8192 // T)), T, **opts)
    opts.pop("router", None)
    model = rng.choice(["paper", "paper", "four"])
    k = rng.choice(CHANNELS[model])
    g = rng.choice([1, 2, 4, 8, 8, 16])
    T = g * _log(rng, max(8, 128 // g), 2048 // g)
    passes = rng.randint(2, 4)
    if kind == "passes":
        B = _log(rng, 1, max(1, (32768 if model == "four" else 8192) // T))
        return _case("passes", model, k, B, T, groups=g, passes=passes, **opts)
    return _case("train", model, k, _log(rng, 1, max(1, 16384 // T)), T, groups=g,
                 passes=passes, n_grad=rng.randint(1, 2), **opts)


def tolerance(case):
    """About four times what the outputs are off from float64 (fp32 sums; bf16 operands and
    results; the bf16 stages that a pass or a gradient chains). The largest single
    difference is that of a channel that nearly cancels in the signed mix."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    if case["kind"] == "train":
        return {"rel": 0.03, "max": 0.5}
    if case["kind"] == "grad":
        return {"rel": 0.02, "max": 0.9}
    if case["kind"] == "passes":
        return {"rel": 0.02, "max": 0.25}
    return {"rel": 0.015, "max": 0.9}


# ------------------------------------------------------------------ inputs

def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _bias(L, k):
    """The paper's initial pattern: alpha[j][l] one-hot."""
    b = torch.zeros(k, L)
    if k == 1:
        b[0, L - 1] = 1
    elif k < L:
        for l in range(L):
            b[l % k, l] = 1
    else:
        for j in range(k):
            b[j, min(j + 1, L - 1)] = 1
    return b.reshape(-1)


def _map(c):
    return [l % c["k"] for l in range(c["L"])]


def _inputs(c, seed):
    """Seeded inputs on the GPU: parameters and the states or embeddings, caches, ..."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _dtype(c)
    L, k, D, Hq, Hkv, d, B, T = (c[n] for n in ("L", "k", "D", "Hq", "Hkv", "d", "B", "T"))
    Lp = (L + c["p"] - 1) // c["p"]
    driver = c["kind"] in ("passes", "train")

    def normal(*shape, std=1.0, mean=0.0, dtype=dt):
        return torch.empty(shape, device="cuda").normal_(mean, std, generator=gen).to(dtype)

    bias = _bias(L, k).cuda()
    if driver or c["router"] == 2:
        bias = bias + 0.2
    P = {
        "g_pre": normal(2, L, D, std=0.1, mean=1.0),
        "W_alpha": normal(2, k * L, Lp * D, std=0.002 if driver else 0.02),
        "b_alpha": torch.stack([bias, bias]).to(dt),
        "g_mid": normal(2, k, D, std=0.1, mean=1.0),
        "Wk": normal(k, Hkv * d, D, std=0.02),
        "Wv": normal(k, Hkv * d, D, std=0.02),
        "g_knorm": normal(k, d, std=0.1, mean=1.0),
        "Kd": normal(k, Hkv, d),
        "Vd": normal(k, Hkv, d),
        "g_in": normal(L, D, std=0.1, mean=1.0),
        "Wq": normal(L, Hq * d, D, std=0.02),
        "g_qnorm": normal(L, d, std=0.1, mean=1.0),
    }
    s = {"P": P}
    if driver:
        s["X"] = normal(B, T, D)
        s["W_o"] = normal(L, D, Hq * d, std=c["out_std"])
        if c["kind"] == "train":
            s["dh_top"] = normal(B, T, D, dtype=torch.float32)
        s["S_cap"] = T
        s["ctx"] = None
        return s
    s["H"] = normal(B, T, L, D)
    s["S_cap"] = (c["ctx"] + T + 63) // 64 * 64
    lo = c["ctx"] // 2 if c["ragged"] else c["ctx"]
    s["ctx"] = torch.randint(lo, c["ctx"] + 1, (B,), generator=gen, device="cuda",
                             dtype=torch.int32)
    shape = (k, B, Hkv, s["S_cap"], d)
    for n in ("Kc", "Vc"):
        s[n] = torch.empty(shape, device="cuda", dtype=dt)
        if c["ctx"]:
            s[n].normal_(generator=gen)
        else:
            s[n].zero_()
    if c["doc_mean"]:
        # A new document starts at each token with probability 1 / mean.
        cut = torch.rand(B, T, generator=gen, device="cuda") < 1.0 / c["doc_mean"]
        at = torch.arange(T, device="cuda", dtype=torch.int64).expand(B, T)
        s["doc"] = torch.cummax(torch.where(cut, at, 0), 1)[0].to(torch.int32).contiguous()
    if c["kind"] == "grad":
        s["dO"] = normal(L, B, T, Hq * d)
    return s


GRADS = wm.PARAM_NAMES


def prepare(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    kind, dt = c["kind"], _dtype(c)
    L, k, B, T, Hq, Hkv, d, D = (c[n] for n in ("L", "k", "B", "T", "Hq", "Hkv", "d", "D"))
    s["kind"], s["L"], s["map"] = kind, L, _map(c)
    s["dims"] = dims = wm.make_dims(
        B, T, L, k, D, Hq, Hkv, d, p=c["p"], S_cap=s["S_cap"], ctx_max=c["ctx"],
        dtype=wm.dtype_code(dt), mix_mode=wm.MIX_SOFTMAX if c["softmax"] else wm.MIX_LINEAR,
        mask_mode=wm.MASK_INCLUSIVE if c["inclusive"] else wm.MASK_PAPER, eps=EPS,
        rope_theta=THETA, router_mode=c["router"], groups=c["groups"])
    params = wm.ParamSet(s["P"])
    if kind in ("step", "layers", "grad"):
        s["O"] = torch.empty((L, B, T, Hq * d), dtype=dt, device="cuda")
    if kind == "step":
        s["ws"] = wm.workspace(dims, wm.OP_LAYER_STEP)
    elif kind == "layers":
        s["ws"] = wm.workspace(dims, wm.OP_LAYER_ATTEND)
        s["ws_pool"] = wm.workspace(dims, wm.OP_POOL)
    elif kind == "pool":
        s["ws"] = wm.workspace(dims, wm.OP_POOL)
    elif kind == "grad":
        wm.layer_step(dims, params, s["H"], s["map"], s["ctx"], s["Kc"], s["Vc"], s["O"])
        s["ws"] = wm.workspace(dims, wm.OP_STEP_BACKWARD)
        s["dKc"] = torch.empty(s["Kc"].shape, device="cuda")
        s["dVc"] = torch.empty(s["Vc"].shape, device="cuda")
        s["dH"] = torch.empty(s["H"].shape, device="cuda")
        s["grads"] = {n: torch.empty(t.shape, device="cuda") for n, t in s["P"].items()}
    elif kind == "passes":
        s["ws"] = wm.workspace(dims, wm.OP_PASSES)
        s["Kc"] = torch.zeros((k, B, Hkv, T, d), dtype=dt, device="cuda")
        s["Vc"] = torch.zeros_like(s["Kc"])
        s["H"] = torch.empty((B, T, L, D), dtype=dt, device="cuda")
        s["h_top"] = torch.empty((B, T, D), dtype=dt, device="cuda")
    else:
        s["passes"], s["n_grad"] = c["passes"], c["n_grad"]
        s["ws"] = torch.empty(wm.passes_backward_workspace(dims, c["n_grad"]),
                              dtype=torch.uint8, device="cuda")
        s["h_top"] = torch.empty((B, T, D), dtype=dt, device="cuda")
        s["dX"] = torch.empty((B, T, D), device="cuda")
        s["dW_o"] = torch.empty(s["W_o"].shape, device="cuda")
        s["grads"] = {n: torch.empty(t.shape, device="cuda") for n, t in s["P"].items()}
    s["passes"], s["n_grad"] = c["passes"], c["n_grad"]
    s["params"] = params
    return s


def run(s):
    kind, dims, params = s["kind"], s["dims"], s["params"]
    if kind == "step":
        wm.layer_step(dims, params, s["H"], s["map"], s["ctx"], s["Kc"], s["Vc"], s["O"],
                      ws=s["ws"], doc_start=s.get("doc"))
        return {"O": s["O"], "Kc": s["Kc"], "Vc": s["Vc"]}
    if kind == "layers":
        for l in range(s["L"]):
            wm.layer_attend(dims, params, l, s["H"], s["map"], s["ctx"], s["Kc"], s["Vc"],
                            s["O"][l], ws=s["ws"])
        wm.pool(dims, params, s["H"], s["ctx"], s["Kc"], s["Vc"], ws=s["ws_pool"])
        return {"O": s["O"], "Kc": s["Kc"], "Vc": s["Vc"]}
    if kind == "pool":
        wm.pool(dims, params, s["H"], s["ctx"], s["Kc"], s["Vc"], ws=s["ws"])
        return {"Kc": s["Kc"], "Vc": s["Vc"]}
    if kind == "passes":
        wm.prefill_passes(dims, params, s["W_o"], s["X"], s["map"], s["passes"], s["Kc"],
                          s["Vc"], s["H"], h_top=s["h_top"], ws=s["ws"])
        return {"H": s["H"], "h_top": s["h_top"], "Kc": s["Kc"], "Vc": s["Vc"]}
    if kind == "grad":
        torch._foreach_zero_([s["dKc"], s["dVc"], s["dH"], *s["grads"].values()])
        wm.layer_step_backward(dims, params, s["H"], s["map"], s["ctx"], s["Kc"], s["Vc"],
                               s["O"], s["dO"], s["dKc"], s["dVc"], s["dH"], s["grads"],
                               ws=s["ws"])
        return {"dH": s["dH"], "dKc": s["dKc"], "dVc": s["dVc"], **s["grads"]}
    torch._foreach_zero_([s["dX"], s["dW_o"], *s["grads"].values()])
    wm.prefill_passes_backward(dims, params, s["W_o"], s["X"], s["map"], s["passes"],
                               s["n_grad"], s["dh_top"], s["dX"], s["dW_o"], s["grads"],
                               h_top=s["h_top"], ws=s["ws"])
    return {"h_top": s["h_top"], "dX": s["dX"], "dW_o": s["dW_o"], **s["grads"]}


# -------------------------------------------------------------------- work

def work(case):
    c = case
    L, k, D, Hq, Hkv, d, B, T, p = (c[n] for n in ("L", "k", "D", "Hq", "Hkv", "d", "B", "T",
                                                   "p"))
    es = 4 if c["dtype"] == "f32" else 2
    N, Lp = B * T, (L + p - 1) // p
    blocks = 0 if c["router"] == 1 else k * L * Lp  # (output, stacked layer) pairs
    if c["router"] == 2:
        blocks = L * sum(1 for j in range(k) for m in range(Lp) if L - 1 - p * m <= j)
    pool = N * (4 * blocks * D + 4 * k * L * D + 4 * k * Hkv * d * D)
    query = N * 2 * L * Hq * d * D
    mean = 0.75 * c["ctx"] if c["ragged"] else c["ctx"]  # ragged contexts: ctx/2 .. ctx
    seen = mean * T + T * (T + 1) / 2
    if c["doc_mean"]:
        seen = min(seen, T * min(float(c["doc_mean"]), T / 2))
    attend = 4 * d * Hq * L * B * seen
    w_pool = es * (2 * blocks * D + 2 * k * Hkv * d * D)
    w_query = es * L * Hq * d * D
    H, O = N * L * D * es, N * L * Hq * d * es
    new, old = 2 * k * N * Hkv * d * es, 2 * k * B * mean * Hkv * d * es
    if c["kind"] in ("step", "layers"):
        return {"bytes": H + w_pool + w_query + old + new + O, "flops": pool + query + attend}
    if c["kind"] == "pool":
        return {"bytes": H + w_pool + new, "flops": pool}
    if c["kind"] == "grad":  # S again, dP, dQ, dK, dV; queries and pool: values, dX, dW
        grads = 2 * (w_pool + w_query)
        return {"bytes": H + 2 * H + 2 * O + new + 2 * new + w_pool + w_query + grads,
                "flops": 2.5 * attend + 3 * (query + pool)}
    block = N * 2 * L * Hq * d * D
    w_o = es * L * D * Hq * d
    flops = (c["passes"] + 1) * pool + c["passes"] * (query + attend + block)
    if c["kind"] == "passes":
        return {"bytes": N * D * es + w_pool + w_query + w_o + H + N * D * es + new,
                "flops": flops}
    flops += c["n_grad"] * (2.5 * attend + 2 * (query + pool + block))
    return {"bytes": N * D * (es + 4 + es + 4) + 3 * (w_pool + w_query + w_o), "flops": flops}


# ----------------------------------------- the same computation in float64

def _rms(x, g):
    return g * x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS)


def _rope(x, pos):
    """x [..., T, d] at positions pos [..., T] (broadcast), rotate-half."""
    d = x.shape[-1]
    f = THETA ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    a = pos.to(torch.float64)[..., None] * f
    x1, x2 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _pool64(c, P, H, pos):
    """K, V rows [k, B, Hkv, T, d] of the tokens H [B, T, L, D] at positions pos [B, T]."""
    L, k, D, Hkv, d = (c[n] for n in ("L", "k", "D", "Hkv", "d"))
    B, T = H.shape[:2]
    sel = [l for l in range(L) if (L - 1 - l) % c["p"] == 0]
    rows = []
    for br in range(2):
        Hn = _rms(H, P["g_pre"][br])
        bias = P["b_alpha"][br].reshape(k, L)
        if c["router"] == 1:
            a = bias.expand(B, T, k, L)
        else:
            W = P["W_alpha"][br].reshape(k, L, len(sel), D)
            if c["router"] == 2:
                keep = torch.tensor([[float(l <= j) for l in sel] for j in range(k)],
                                    device=H.device, dtype=H.dtype)
                W = W * keep[:, None, :, None]
            x = Hn[:, :, sel].reshape(B * T, -1)
            a = (x @ W.reshape(k * L, -1).t()).reshape(B, T, k, L) + bias
        if c["router"] == 2:
            low = torch.ones(k, L, device=H.device, dtype=torch.bool).tril()
            a = a.masked_fill(~low, -math.inf if c["softmax"] else 0.0)
        if c["softmax"]:
            a = torch.softmax(a, -1)
        mixed = torch.matmul(a, Hn)  # [B, T, k, D]
        u = _rms(mixed, P["g_mid"][br]).permute(2, 0, 1, 3).reshape(k, B * T, D)
        y = torch.bmm(u, P["Wk" if br == 0 else "Wv"].transpose(1, 2).contiguous())
        y = y.reshape(k, B, T, Hkv, d).permute(0, 1, 3, 2, 4)
        if br == 0:
            y = _rope(_rms(y, P["g_knorm"][:, None, None, None, :]), pos[None, :, None])
        rows.append(y)
    return rows


def _query64(c, P, l, h, pos):
    """Queries [B, Hq, T, d] of layer l for h [B, T, D]."""
    q = _rms(h, P["g_in"][l]) @ P["Wq"][l].t()
    q = q.reshape(*h.shape[:2], c["Hq"], c["d"]).transpose(1, 2)
    return _rope(_rms(q, P["g_qnorm"][l]), pos[:, None])


def _attend_rows(q, K, V, kd, vd, pos, first, inclusive):
    """q [b, Hq, T, d], K and V [b, Hkv, S, d], pos and first [b, T]: [b, Hq, T, d]."""
    nb, Hq, T, d = q.shape
    Hkv, S = K.shape[1:3]
    g = Hq // Hkv
    qs = q.reshape(nb * Hkv, g * T, d) / math.sqrt(d)
    sc = torch.bmm(qs, K.reshape(nb * Hkv, S, d).transpose(1, 2).contiguous())
    slot = torch.arange(S, device=q.device)
    at, low = pos[..., None], first[..., None]
    see = ((slot <= at) if inclusive else (slot < at)) & (slot >= low)
    sc = sc.reshape(nb, Hkv, g, T, S).masked_fill(~see[:, None, None], -math.inf)
    if not inclusive:
        sd = torch.matmul(qs.reshape(nb, Hkv, g * T, d), kd[:, :, None])
        sc = torch.cat([sc, sd.reshape(nb, Hkv, g, T, 1)], -1)
    w = torch.softmax(sc, -1)
    o = torch.bmm(w[..., :S].reshape(nb * Hkv, g * T, S), V.reshape(nb * Hkv, S, d))
    o = o.reshape(nb, Hkv, g, T, d)
    if not inclusive:
        o = o + w[..., S:] * vd[:, None, None, :]
    return o.reshape(nb, Hq, T, d)


def _attend64(c, P, l, q, K, V, pos, first, grad=False):
    """Consumer l over K, V [B, Hkv, S, d]: [B, T, Hq * d], a block of rows at a time."""
    j, dt = l % c["k"], torch.float64
    B, Hq, T = q.shape[:3]
    step = min(T, 512)
    nb = max(1, min(B, (1 << 27) // (Hq * step * (c["ctx"] + c["T"]))))
    outs = []
    for b in range(0, B, nb):
        part = []
        for t in range(0, T, step):
            at = pos[b:b + nb, t:t + step]
            S = min(int(at.max()) + 1, K.shape[2])
            args = (q[b:b + nb, :, t:t + step], K[b:b + nb, :, :S].to(dt),
                    V[b:b + nb, :, :S].to(dt), P["Kd"][j], P["Vd"][j], at,
                    first[b:b + nb, t:t + step], c["inclusive"])
            part.append(checkpoint(_attend_rows, *args, use_reentrant=False) if grad
                        else _attend_rows(*args))
        outs.append(torch.cat(part, 2))
    return torch.cat(outs).transpose(1, 2).reshape(B, T, -1)


def _put(cache, rows, pos):
    """cache [k, B, Hkv, S, d] with rows at slots pos [B, T] (a new tensor)."""
    ix = pos.long()[None, :, None, :, None].expand(rows.shape)
    return cache.scatter(3, ix, rows.to(cache.dtype))


def _passes64(c, P, W_o, X, n_cut):
    """The fixed-point passes; the cache entering pass n_cut (0-based) is detached (none:
    n_cut = 0). Returns states [B, T, L, D], the top state and the caches."""
    L, g, B, T = c["L"], c["groups"], c["B"], c["T"]
    every = torch.arange(T, device=X.device).expand(B, T)
    first = torch.zeros_like(every)
    with torch.set_grad_enabled(torch.is_grad_enabled() and n_cut == 0):
        K, V = _pool64(c, P, X[:, :, None].expand(B, T, L, -1), every)
    groups = [every[:, q::g] for q in range(g)]
    states, tops = [None] * g, [None] * g
    wanted = torch.is_grad_enabled()
    for n in range(c["passes"]):
        with torch.set_grad_enabled(wanted and n >= n_cut):
            for q, pos in enumerate(groups):
                h, hs = X[:, q::g], []
                for l in range(L):
                    hs.append(h)
                    Q = _query64(c, P, l, h, pos)
                    o = _attend64(c, P, l, Q, K[l % c["k"]], V[l % c["k"]], pos,
                                  first[:, q::g], torch.is_grad_enabled())
                    h = h + o @ W_o[l].t()
                states[q], tops[q] = torch.stack(hs, 2), h
                if n + 1 < c["passes"] or q + 1 < g or not wanted:
                    Kn, Vn = _pool64(c, P, states[q], pos)
                    K, V = _put(K, Kn, pos), _put(V, Vn, pos)
    H = torch.stack(states, 2).reshape(B, T, L, -1)
    return H, torch.stack(tops, 2).reshape(B, T, -1), K, V


def exact(case, seed):
    c, s = dict(case), _inputs(case, seed)
    kind, L, B, T = c["kind"], c["L"], c["B"], c["T"]
    grad = kind in ("grad", "train")
    P = {n: t.double().requires_grad_(grad) for n, t in s["P"].items()}
    if kind in ("passes", "train"):
        X, W_o = s["X"].double().requires_grad_(grad), s["W_o"].double().requires_grad_(grad)
        if kind == "passes":
            with torch.no_grad():
                H, top, K, V = _passes64(c, P, W_o, X, 0)
            return {"H": H, "h_top": top, "Kc": K, "Vc": V}
        cut = c["passes"] - c["n_grad"]
        _, top, _, _ = _passes64(c, P, W_o, X, cut)
        leaves = [X, W_o, *P.values()]
        got = torch.autograd.grad(top, leaves, s["dh_top"].double(), allow_unused=True)
        got = [torch.zeros_like(x) if y is None else y for x, y in zip(leaves, got)]
        return {"h_top": top.detach(), "dX": got[0], "dW_o": got[1],
                **dict(zip(P, got[2:]))}
    pos = s["ctx"][:, None].long() + torch.arange(T, device="cuda")
    first = s["doc"].long() if "doc" in s else torch.zeros_like(pos)
    H = s["H"].double().requires_grad_(grad)
    with torch.set_grad_enabled(grad):
        Kn, Vn = _pool64(c, P, H, pos)
    if not grad:
        out = {"Kc": _put(s["Kc"].double(), Kn, pos), "Vc": _put(s["Vc"].double(), Vn, pos)}
        if kind == "pool":
            return out
        O = torch.empty((L, B, T, c["Hq"] * c["d"]), device="cuda", dtype=torch.float64)
        for l in range(L):
            Q = _query64(c, P, l, H[:, :, l], pos)
            O[l] = _attend64(c, P, l, Q, out["Kc"][l % c["k"]], out["Vc"][l % c["k"]], pos,
                             first)
        return {"O": O, **out}
    # Gradients: each consumer's attention on detached rows, then one walk through the pool.
    Kl, Vl = Kn.detach().requires_grad_(), Vn.detach().requires_grad_()
    dK, dV = torch.zeros_like(Kl), torch.zeros_like(Vl)
    leaves = [H, *P.values()]
    total = [torch.zeros_like(x) for x in leaves]
    for l in range(L):
        j = l % c["k"]
        Kj, Vj = Kl[j].detach().requires_grad_(), Vl[j].detach().requires_grad_()
        Q = _query64(c, P, l, H[:, :, l], pos)
        o = _attend64(c, P, l, Q, Kj, Vj, pos, first, True)
        got = torch.autograd.grad(o, [Kj, Vj, *leaves], s["dO"][l].double(),
                                  allow_unused=True)
        dK[j] += got[0]
        dV[j] += got[1]
        for a, b in zip(total, got[2:]):
            if b is not None:
                a += b
    got = torch.autograd.grad([Kn, Vn], leaves, [dK, dV], allow_unused=True)
    for a, b in zip(total, got):
        if b is not None:
            a += b
    cache = torch.zeros(s["Kc"].shape, device="cuda", dtype=torch.float64)
    return {"dH": total[0], "dKc": _put(cache, dK, pos), "dVc": _put(cache, dV, pos),
            **dict(zip(P, total[1:]))}
