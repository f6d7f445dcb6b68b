"""Timed workloads of the draft/verify hot path, through its public entry points.

A case is a dict of plain values; ``prepare`` builds what a serving program
holds before the call (weights, expert tables, workspaces, input rows),
``run`` makes one pass and returns every output, ``exact`` gives the same
outputs in 64 bits from plain torch.

Kinds:
  verify   ``de_verify_layer``: one target MoE layer over a block of T
           positions (Eq. 4), with the residual + RMSNorm epilogue of a stack;
  draft    ``de_draft_layer_topr``: one drafter layer (Eq. 5);
  dense    ``de_dense_swiglu``: the dense layer 0 of the stack;
  head     ``de_lm_head`` and ``de_accept_len``: logits and acceptance of a block;
  model    ``DeviceModel.forward``: a whole stack, target or drafter, to logits;
  distill  ``DeviceModel.distill``: the self-distillation signals of a block.

A layer case holds ``layers`` layers' weights and calls each once, as a stack
does (with attention between them, so that each has its own input rows): a
program never meets the same layer twice in a row, and a single layer's few
read weights would stay in the last-level cache from pass to pass.
"""
import math

import torch

import paper_2607_24434_amd as de

DTYPES = {"f32": de.DE_F32, "bf16": de.DE_BF16, "q4": de.DE_Q4_0}
EPS = 1e-6
# The DeepSeek-V2-Lite-shaped layer: 64 routed experts, top-6, two shared
# experts as one block, one draft expert.
V2 = dict(hidden=2048, experts=64, top_k=6, inter=1408, shared=2816, draft=1408,
          score="softmax", norm_topk=False, wdtype="bf16", router_std=0.1)
# The same sizes with a sigmoid router, a selection bias and renormalised gates.
MOONLIGHT = dict(V2, score="sigmoid", norm_topk=True, router_std=0.02)
VOCAB = 102400
DENSE = 10944


def listed():
    return [
        # The smallest call: a tiny fp32 layer over 5 positions. Latency and launches only.
        dict(name="verify-5-tiny-f32", kind="verify", layers=1, positions=5, hidden=256, experts=8,
             top_k=2, inter=128, shared=128, draft=64, score="softmax", norm_topk=True,
             wdtype="f32", router_std=0.02),
        # One drafted token: the drafter's layers at a single position.
        dict(V2, name="draft-1", kind="draft", layers=6, positions=1, topr=1, with_draft=True),
        # The same with the 4.5-bit expert weights of small devices.
        dict(V2, name="draft-1-q4", kind="draft", layers=6, positions=1, topr=1, with_draft=True,
             wdtype="q4"),
        # The ordinary verify block: 8 drafts and the last committed token.
        dict(V2, name="verify-9", kind="verify", layers=2, positions=9),
        # The same with 4.5-bit expert weights.
        dict(V2, name="verify-9-q4", kind="verify", layers=3, positions=9, wdtype="q4"),
        # The long verify block (16 drafts) on the sigmoid router.
        dict(MOONLIGHT, name="verify-17-sigmoid", kind="verify", layers=2, positions=17),
        # The largest block: every expert is read, popular ones for many positions.
        dict(V2, name="verify-64", kind="verify", layers=1, positions=64),
        # The dense layer 0 of the stack over an ordinary block.
        dict(name="dense-9", kind="dense", positions=9, hidden=2048, inter=DENSE, wdtype="bf16"),
        # Logits and acceptance of a long block.
        dict(name="head-17", kind="head", positions=17, hidden=2048, vocab=VOCAB),
        # A drafted token through a stack: embedding, dense layer, MoE layers, head, argmax.
        dict(V2, name="model-draft-1", kind="model", layers=4, positions=1, mode="draft",
             vocab=VOCAB, dense=DENSE),
        # A verify block through the same stack.
        dict(V2, name="model-verify-9", kind="model", layers=4, positions=9, mode="target",
             vocab=VOCAB, dense=DENSE),
        # Signals for training the draft experts over a batch of positions.
        dict(V2, name="distill-32", kind="distill", layers=2, positions=32, vocab=VOCAB,
             dense=DENSE, tau=2.0),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of ``step`` in [lo, hi], spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["verify"] * 5 + ["draft"] * 3 + ["dense", "head", "model", "model"])
    step = rng.choice([8, 32, 256])
    hidden = _log(rng, 512, 2048, step)
    if kind == "head":
        return dict(kind=kind, positions=_log(rng, 1, 64), hidden=hidden,
                    vocab=_log(rng, 1000, VOCAB))
    if kind == "dense":
        return dict(kind=kind, positions=_log(rng, 1, 64), hidden=hidden,
                    inter=_log(rng, 256, DENSE, step), wdtype="bf16")
    q4 = rng.random() < 0.25
    if q4:
        step = max(step, 32)
        hidden = max(512, hidden // 32 * 32)
    inter = _log(rng, 128, 1408, min(step, 128))
    experts = rng.choice([8, 16, 33, 60, 64, 128])
    while experts * inter * hidden > 64 * 1408 * 2048:
        experts = experts // 2
    sigmoid = rng.random() < 0.4
    c = dict(kind=kind, hidden=hidden, experts=experts, top_k=rng.choice([2, 4, 6, 8]),
             inter=inter, shared=rng.choice([0, 1, 2]) * inter,
             draft=inter, score="sigmoid" if sigmoid else "softmax",
             norm_topk=rng.random() < 0.5, wdtype="q4" if q4 else "bf16",
             router_std=0.02 if sigmoid else 0.1)
    if kind == "draft":
        r = rng.choice([1, 1, 1, 2, 3])
        c.update(layers=rng.choice([2, 4, 6]), positions=rng.choice([1, 1, _log(rng, 2, 16)]),
                 topr=min(r, c["top_k"]), with_draft=r == 1)
    elif kind == "verify":
        c.update(layers=rng.choice([1, 2]), positions=_log(rng, 1, 64))
    else:
        mode = rng.choice(["target", "draft"])
        c.update(layers=rng.choice([1, 2, 3]), mode=mode, dense=_log(rng, 256, DENSE, 8),
                 positions=1 if mode == "draft" else _log(rng, 1, 33),
                 vocab=_log(rng, 1000, VOCAB))
    return c


# ---------------------------------------------------------------- inputs


def _normal(gen, shape, std, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _q4_pack(w, out):
    """Q4_0 blocks of the weights w [n, rows * cols] into out [n, bytes]: 32
    weights share d = extreme / -8, code = round(w / d) + 8."""
    n = w.shape[0]
    b = w.view(n, -1, 32)
    at = b.abs().argmax(dim=2, keepdim=True)
    d = (b.gather(2, at) / -8.0).half()
    q = (b / d.float() + 8.5).floor_().clamp_(0, 15).to(torch.uint8)
    codes = q[:, :, :16] | (q[:, :, 16:] << 4)
    nc = codes.shape[1] * 16
    out[:, :nc] = codes.reshape(n, nc)
    out[:, nc:] = d.reshape(n, -1).view(torch.uint8)


def _blocks(gen, n, inter, hidden, wdtype):
    """n expert blocks [G | U | D] of weights N(0, 0.02), one per row."""
    if wdtype == "q4":
        m = inter * hidden
        mb = m * 9 // 16
        out = torch.empty(n, 3 * mb, dtype=torch.uint8, device="cuda")
        for part in range(3):
            for e in range(0, n, 16):
                k = min(16, n - e)
                _q4_pack(_normal(gen, (k, m), 0.02), out[e:e + k, part * mb:(part + 1) * mb])
        return out
    dt = torch.float32 if wdtype == "f32" else torch.bfloat16
    return _normal(gen, (n, 3 * inter * hidden), 0.02, dt)


def _desc(c):
    return de.make_desc(c["hidden"], c["experts"], c["top_k"], c["inter"], c["shared"], c["draft"],
                        de.DE_SIGMOID if c["score"] == "sigmoid" else de.DE_SOFTMAX,
                        c["norm_topk"], 1.0, DTYPES[c["wdtype"]])


def _layer_weights(c, gen):
    H, N = c["hidden"], c["experts"]
    w = dict(router=_normal(gen, (N, H), c["router_std"]),
             bias=_normal(gen, (N,), 0.1) if c["score"] == "sigmoid" else None,
             routed=_blocks(gen, N, c["inter"], H, c["wdtype"]), shared=None, draft=None)
    if c["shared"]:
        w["shared"] = _blocks(gen, 1, c["shared"], H, c["wdtype"])[0]
    if c["draft"]:
        w["draft"] = _blocks(gen, 1, c["draft"], H, c["wdtype"])[0]
    return w


def _inputs(c, seed):
    """Everything random of a case, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    T, H = c["positions"], c["hidden"]
    if c["kind"] in ("verify", "draft"):
        L = c["layers"]
        return dict(layers=[_layer_weights(c, gen) for _ in range(L)],
                    x=_normal(gen, (L, T, H), 1.0), residual=_normal(gen, (L, T, H), 1.0))
    if c["kind"] == "dense":
        return dict(w=_blocks(gen, 1, c["inter"], H, c["wdtype"])[0],
                    x=_normal(gen, (T, H), 1.0), residual=_normal(gen, (T, H), 1.0))
    if c["kind"] == "head":
        V = c["vocab"]
        return dict(x=_normal(gen, (T, H), 1.0), lm=_normal(gen, (V, H), 0.02, torch.bfloat16),
                    drafts=torch.randint(0, V, (max(1, T - 1),), generator=gen, device="cuda",
                                         dtype=torch.int32))
    V = c["vocab"]
    return dict(layers=[_layer_weights(c, gen) for _ in range(c["layers"])],
                emb=_normal(gen, (V, H), 1.0, torch.bfloat16),
                lm=_normal(gen, (V, H), 0.02, torch.bfloat16),
                dense=_blocks(gen, 1, c["dense"], H, "bf16")[0],
                tokens=torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32))


def prepare(case, seed):
    c = case
    s = dict(_inputs(c, seed), case=c)
    T, H = c["positions"], c["hidden"]

    def empty(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if c["kind"] in ("verify", "draft"):
        L, k = c["layers"], c["top_k"]
        s["desc"] = _desc(c)
        stride = de.expert_bytes(DTYPES[c["wdtype"]], c["inter"], H)
        s["tables"] = [de.make_table(w["routed"], stride, None, c["experts"]) for w in s["layers"]]
        s["y"], s["normed"] = empty(L, T, H), empty(L, T, H)
        s["epi"] = [de.make_epilogue(s["residual"][i], s["normed"][i], EPS) for i in range(L)]
        s["idx"], s["gate"] = empty(L, T, k, dtype=torch.int32), empty(L, T, k)
        s["n_union"] = empty(L, 1, dtype=torch.int32)
        s["ws"] = de.workspace(s["desc"], T)
        s["calls"] = [dict(w=w, x=s["x"][i], y=s["y"][i], idx=s["idx"][i], gate=s["gate"][i],
                           n_union=s["n_union"][i], epi=s["epi"][i], table=s["tables"][i])
                      for i, w in enumerate(s["layers"])]
    elif c["kind"] == "dense":
        s["y"], s["normed"] = empty(T, H), empty(T, H)
        s["epi"] = de.make_epilogue(s["residual"], s["normed"], EPS)
        s["ws"] = torch.empty(de.de_dense_workspace_bytes(T, H, c["inter"]), dtype=torch.uint8,
                              device="cuda")
    elif c["kind"] == "head":
        s["logits"] = empty(T, c["vocab"])
        s["argmax"], s["out"] = empty(T, dtype=torch.int32), empty(2, dtype=torch.int32)
        s["ws"] = de.accept_workspace(T - 1, c["vocab"])
    else:
        V, L = c["vocab"], c["layers"]
        s["model"] = de.DeviceModel(_desc(c), s["layers"], V, s["emb"], s["lm"], s["dense"],
                                    c["dense"], de.DE_BF16, EPS, 1.0, T)
        if c["kind"] == "model":
            s["logits"], s["argmax"] = empty(T, V), empty(T, dtype=torch.int32)
            s["n_union"] = empty(L, dtype=torch.int32) if c["mode"] == "target" else None
        else:
            s["m_star"], s["router_kl"] = empty(L, T, H), empty(L, T)
            s["logit_kl"], s["token_ce"] = empty(T), empty(T)
    return s


def run(state):
    s, c = state, state["case"]
    T = c["positions"]
    if c["kind"] == "verify":
        for a in s["calls"]:
            w = a["w"]
            de.de_verify_layer(s["desc"], T, a["x"], w["router"], w["bias"], a["table"],
                               w["shared"], a["y"], topk_idx=a["idx"], topk_gate=a["gate"],
                               n_union=a["n_union"], ws=s["ws"], epi=a["epi"])
        return dict(y=s["y"], normed=s["normed"], idx=s["idx"], gate=s["gate"],
                    n_union=s["n_union"])
    if c["kind"] == "draft":
        for a in s["calls"]:
            w = a["w"]
            de.de_draft_layer_topr(s["desc"], T, a["x"], w["router"], w["bias"], a["table"],
                                   w["shared"], w["draft"] if c["with_draft"] else None, 1.0,
                                   c["topr"], a["y"], a["idx"], a["gate"], s["ws"], epi=a["epi"])
        return dict(y=s["y"], normed=s["normed"], idx=s["idx"], gate=s["gate"])
    if c["kind"] == "dense":
        de.de_dense_swiglu(T, c["hidden"], c["inter"], DTYPES[c["wdtype"]], s["x"], s["w"], s["y"],
                           s["ws"], epi=s["epi"])
        return dict(y=s["y"], normed=s["normed"])
    if c["kind"] == "head":
        de.de_lm_head(T, c["hidden"], c["vocab"], s["x"], s["lm"], s["logits"])
        de.de_accept_len(T - 1, c["vocab"], s["logits"], s["drafts"] if T > 1 else None,
                         s["argmax"], s["out"], s["ws"])
        return dict(logits=s["logits"], argmax=s["argmax"], out=s["out"])
    if c["kind"] == "model":
        s["model"].forward(s["tokens"], de.DE_TARGET if c["mode"] == "target" else de.DE_DRAFT,
                           s["logits"], s["argmax"], s["n_union"])
        return dict(logits=s["logits"], argmax=s["argmax"], n_union=s["n_union"])
    s["model"].distill(s["tokens"], c["tau"], s["m_star"], s["router_kl"], s["logit_kl"],
                       s["token_ce"])
    return dict(m_star=s["m_star"], router_kl=s["router_kl"], logit_kl=s["logit_kl"],
                token_ce=s["token_ce"])


# ---------------------------------------------------------------- what a pass cannot do without


def _layer_work(c, T, entries, draft):
    """Bytes and operations of one layer whose positions use `entries` routed experts each."""
    H, N = c["hidden"], c["experts"]
    k = min(c["top_k"], N)
    union = N * (1.0 - (1.0 - entries / N) ** T)  # expected under even routing
    ew = de.expert_bytes(DTYPES[c["wdtype"]], 1, H)  # bytes per intermediate row of G, U and D
    rows = union * c["inter"] + c["shared"] + draft
    b = rows * ew + N * H * 4 + 4 * T * H * 4 + T * k * 8
    f = 2.0 * T * N * H + 6.0 * T * H * (entries * c["inter"] + c["shared"] + draft)
    return b, f


def work(case):
    c = case
    T, H = c["positions"], c["hidden"]
    if c["kind"] == "verify":
        b, f = _layer_work(c, T, c["top_k"], 0)
        return dict(bytes=c["layers"] * b, flops=c["layers"] * f)
    if c["kind"] == "draft":
        b, f = _layer_work(c, T, c["topr"], c["draft"] if c["with_draft"] else 0)
        return dict(bytes=c["layers"] * b, flops=c["layers"] * f)
    if c["kind"] == "dense":
        w = de.expert_bytes(DTYPES[c["wdtype"]], c["inter"], H)
        return dict(bytes=w + 4 * T * H * 4, flops=6.0 * T * H * c["inter"])
    V = c["vocab"]
    if c["kind"] == "head":
        return dict(bytes=V * H * 2 + T * H * 4 + T * V * 4, flops=2.0 * T * V * H)

    def stack(mode):
        if mode == "target":
            b, f = _layer_work(c, T, c["top_k"], 0)
        else:
            b, f = _layer_work(c, T, 1, c["draft"])
        b, f = c["layers"] * b, c["layers"] * f
        b += de.expert_bytes(de.DE_BF16, c["dense"], H) + V * H * 2 + T * V * 4 + T * H * 2
        return b, f + 6.0 * T * H * c["dense"] + 2.0 * T * V * H

    if c["kind"] == "model":
        b, f = stack(c["mode"])
        return dict(bytes=b, flops=f)
    (b1, f1), (b2, f2) = stack("target"), stack("draft")
    return dict(bytes=b1 + b2, flops=f1 + f2)


def tolerance(case):
    """Activations, products and sums are fp32 whatever the weights' format.
    Against 64 bits a layer's outputs are off by up to 3.5e-7 and a stack's
    logits by 6e-7: another order of the sums stays within four times that.
    The logit divergence is a small difference of sums over the vocabulary
    and is off by 6e-5."""
    if case["kind"] == "distill":
        return {"rel": 2.5e-4, "max": 2e-3}
    if case["kind"] == "model":
        return {"rel": 3e-6, "max": 6e-5}
    return {"rel": 2e-6, "max": 4e-5}


# ---------------------------------------------------------------- the same in 64 bits


def _mats(block, inter, hidden, wdtype):
    """(G [I, H], U [I, H], D [H, I]) of one block in 64 bits."""
    m = inter * hidden
    if wdtype == "q4":
        mb = m * 9 // 16
        parts = []
        for i in range(3):
            raw = block[i * mb:(i + 1) * mb]
            codes = raw[:m // 2].view(-1, 16)
            q = torch.cat([codes & 15, codes >> 4], dim=1).double() - 8.0
            d = raw[m // 2:].clone().view(torch.float16).double()
            parts.append((q * d[:, None]).reshape(-1))
    else:
        parts = [p.double() for p in block.view(3, m)]
    return (parts[0].view(inter, hidden), parts[1].view(inter, hidden),
            parts[2].view(hidden, inter))


def _swiglu(x, block, inter, hidden, wdtype):
    g, u, d = _mats(block, inter, hidden, wdtype)
    a = x @ g.t()
    return (a * torch.sigmoid(a) * (x @ u.t())) @ d.t()


def _rmsnorm(h):
    return h / torch.sqrt(h.square().mean(dim=-1, keepdim=True) + EPS)


def _routing(c, w, x):
    """Router logits, the ordered top-k experts and their gates."""
    z = x @ w["router"].double().t()
    b = w["bias"].double() if w["bias"] is not None else 0.0
    if c["score"] == "sigmoid":
        score = torch.sigmoid(z)
        key = score + b
    else:
        key = z + b
        score = torch.softmax(key, dim=-1)
    idx = key.topk(c["top_k"], dim=-1).indices
    gate = score.gather(1, idx)
    if c["norm_topk"]:
        gate = gate / gate.sum(dim=-1, keepdim=True)
    return z, idx, gate


def _moe(c, w, x, entries, with_draft):
    """One layer over rows x: output, logits, gates and each routed term by rank."""
    H = c["hidden"]
    z, idx, gate = _routing(c, w, x)
    y = torch.zeros_like(x)
    if c["shared"]:
        y += _swiglu(x, w["shared"], c["shared"], H, c["wdtype"])
    lower = torch.zeros_like(x)  # the routed terms below the leading expert
    for e in torch.unique(idx[:, :entries]).tolist():
        t, j = (idx[:, :entries] == e).nonzero(as_tuple=True)
        o = _swiglu(x[t], w["routed"][e], c["inter"], H, c["wdtype"]) * gate[t, j][:, None]
        y.index_add_(0, t, o)
        lower.index_add_(0, t, o * (j > 0)[:, None])
    if with_draft and w["draft"] is not None:
        y += _swiglu(x, w["draft"], c["draft"], H, c["wdtype"])
    return y, z, gate, lower


def _head(x, lm):
    return torch.cat([x @ p.double().t() for p in lm.split(16384)], dim=1)


def _stack(c, s, mode):
    """Logits [T, V], the layers' router logits and lower-ranked routed terms."""
    h = s["emb"][s["tokens"].long()].double()
    h = h + _swiglu(_rmsnorm(h), s["dense"], c["dense"], c["hidden"], "bf16")
    zs, lows = [], []
    for w in s["layers"]:
        target = mode == "target"
        y, z, _, low = _moe(c, w, _rmsnorm(h), c["top_k"] if target else 1, not target)
        h = h + y
        zs.append(z)
        lows.append(low)
    return _head(_rmsnorm(h), s["lm"]), zs, lows


def _kl(a, b):
    la, lb = torch.log_softmax(a, -1), torch.log_softmax(b, -1)
    return (la.exp() * (la - lb)).sum(-1)


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    if c["kind"] in ("verify", "draft"):
        ys, gates = [], []
        entries = c["top_k"] if c["kind"] == "verify" else c["topr"]
        for i, w in enumerate(s["layers"]):
            y, _, gate, _ = _moe(c, w, s["x"][i].double(), entries,
                                 c["kind"] == "draft" and c["with_draft"])
            ys.append(y + s["residual"][i].double())
            gates.append(gate)
        y = torch.stack(ys)
        r = dict(y=y, normed=_rmsnorm(y), idx=None, gate=torch.stack(gates))
        return dict(r, n_union=None) if c["kind"] == "verify" else r
    if c["kind"] == "dense":
        y = s["residual"].double() + _swiglu(s["x"].double(), s["w"], c["inter"], c["hidden"],
                                             c["wdtype"])
        return dict(y=y, normed=_rmsnorm(y))
    if c["kind"] == "head":
        return dict(logits=_head(s["x"].double(), s["lm"]), argmax=None, out=None)
    if c["kind"] == "model":
        return dict(logits=_stack(c, s, c["mode"])[0], argmax=None, n_union=None)
    lt, zt, low = _stack(c, s, "target")
    ld, zd, _ = _stack(c, s, "draft")
    tau = c["tau"]
    ce = -torch.log_softmax(ld, -1).gather(1, lt.argmax(-1, keepdim=True))[:, 0]
    return dict(m_star=torch.stack(low), router_kl=torch.stack([_kl(a, b) for a, b in zip(zt, zd)]),
                logit_kl=tau * tau * _kl(lt / tau, ld / tau), token_ce=ce)
