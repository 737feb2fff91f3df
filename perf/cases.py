"""Performance cases of the EAT MoE layer: what a program that uses this
package has it do, at the sizes it does it.

Three kinds of call, each through the package's public objects:

  * ``layer``: one MoE-layer forward (``EatLayer.forward``) -- a decode step,
    a mixed batch of a few hundred tokens, or a prefill chunk -- in the three
    routing modes, on packed and on row-major weights (the default layout);
  * ``stack``: one decode step through stacked layers (``EatStack.forward``);
  * ``ppl``: one token per sequence through the LM head for the perplexity
    signal of the threshold (``PplSignal.step``).

Layer shapes are those of ``workload.SHAPES``.  Inputs follow the same recipe
(clustered Gaussian hidden states, N(0, 1/fan-in) weights), drawn on the GPU.
EAT layers start from the account state a running model has: every expert
has been used, and its C_s is near its output norm.

``exact`` is the same computation in 64 bits in plain torch.
"""
import math

import torch

from paper_2609_33614_amd import _lib as L
from paper_2609_33614_amd.layer import EatLayer, EatStack, PplSignal, pack_weights
from workload import SHAPES

DEV = "cuda"
EPS = 1e-6            # RMSNorm epsilon of the stacked layers

# largest calls the drawn cases make per shape: no costlier than the largest listed case
MAX_TOKENS = {"tiny": 512, "mixtral": 1024, "finegrained": 4096, "shared": 6144, "qwen3": 4096}
# experts a token selects under Top-P (p = 0.6) on these inputs, for work()
TOPP_K = {"tiny": 1.3, "mixtral": 1.3, "finegrained": 6.7, "shared": 6.5, "qwen3": 11.0}


def listed():
    def layer(name, shape, tokens, mode, packed, trend=False, share=False):
        return {"name": name, "kind": "layer", "shape": shape, "tokens": tokens, "mode": mode,
                "packed": packed, "trend": trend, "share": share}

    return [
        # the smallest call: the fp32 layer of the correctness runs, a small
        # batch; launches and latency are all there is
        layer("tiny_fp32_32_eat", "tiny", 32, "eat", False, trend=True),
        # a single user's decode step on big experts
        layer("mixtral_decode_1_eat", "mixtral", 1, "eat", True, trend=True),
        # the headline decode batch
        layer("mixtral_decode_64_eat", "mixtral", 64, "eat", True, trend=True),
        # an odd batch on weights as a checkpoint holds them, baseline routing
        layer("mixtral_decode_37_topk_rows", "mixtral", 37, "topk", False),
        # a mixed batch (decode tokens and prompt chunks together) under the
        # share reading of C_s, which keeps all experts in use
        layer("mixtral_mixed_500_eat_share", "mixtral", 500, "eat", True, trend=True, share=True),
        # a large serving batch on many small experts
        layer("finegrained_decode_256_eat", "finegrained", 256, "eat", True, trend=True),
        # a mixed batch of odd size over 128 experts, row-major weights
        layer("qwen3_mixed_1000_topk_rows", "qwen3", 1000, "topk", False),
        # a prefill chunk on many small experts
        layer("finegrained_prefill_4096_topk", "finegrained", 4096, "topk", True),
        # decode with an always-on expert, the nucleus baseline, row-major
        layer("shared_decode_128_topp_rows", "shared", 128, "topp", False),
        # the largest prefill chunk, always-on expert
        layer("shared_prefill_8192_eat", "shared", 8192, "eat", True),
        # a whole model's MoE layers for one decode step
        {"name": "stack16_decode_64_eat", "kind": "stack", "layers": 16, "tokens": 64, "mode": "eat", "packed": True},
        # the perplexity signal of a decode batch
        {"name": "ppl_64", "kind": "ppl", "sequences": 64, "d": 4096, "vocab": 32000},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    u = rng.random()
    if u < 0.10:
        return {"kind": "ppl", "sequences": _log_int(rng, 1, 256), "d": rng.choice([2048, 4096]),
                "vocab": 64 * rng.randint(250, 800)}
    if u < 0.20:
        return {"kind": "stack", "layers": rng.randint(2, 16), "tokens": _log_int(rng, 1, 64), "mode": "eat",
                "packed": rng.random() < 0.5}
    shape = rng.choice(["tiny", "mixtral", "mixtral", "finegrained", "finegrained", "shared", "qwen3"])
    mode = rng.choice(["eat", "eat", "topk", "topp"])
    most = MAX_TOKENS[shape] if mode != "topp" else min(1024, MAX_TOKENS[shape])
    return {"kind": "layer", "shape": shape, "tokens": _log_int(rng, 1, most), "mode": mode,
            "packed": shape != "tiny" and rng.random() < 0.5, "trend": mode == "eat" and rng.random() < 0.5,
            "share": mode == "eat" and rng.random() < 0.3}


# ------------------------------------------------------------------ inputs --

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + stream)
    return g


def _normal(gen, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)


def _weights(s, seed, stream):
    dt = torch.bfloat16 if s.bf16 else torch.float32
    g = _gen(seed, stream)
    w = {"w_router": _normal(g, (s.E, s.d), s.d ** -0.5, torch.float32),
         "w1": _normal(g, (s.E, s.F, s.d), s.d ** -0.5, dt),
         "w3": _normal(g, (s.E, s.F, s.d), s.d ** -0.5, dt),
         "w2": _normal(g, (s.E, s.d, s.F), s.F ** -0.5, dt)}
    if s.F_shared:
        w["ws1"] = _normal(g, (s.F_shared, s.d), s.d ** -0.5, dt)
        w["ws3"] = _normal(g, (s.F_shared, s.d), s.d ** -0.5, dt)
        w["ws2"] = _normal(g, (s.d, s.F_shared), s.F_shared ** -0.5, dt)
    return w


def _hidden(s, T, seed, stream):
    """Clustered hidden states: x = mu_c + N(0, I), mu_c ~ N(0, 2 I)."""
    g = _gen(seed, stream)
    mu = _normal(g, (s.clusters, s.d), math.sqrt(2.0), torch.float32)
    c = torch.randint(0, s.clusters, (T,), device=DEV, generator=g)
    x = mu[c] + _normal(g, (T, s.d), 1.0, torch.float32)
    return x.to(torch.bfloat16 if s.bf16 else torch.float32).contiguous()


def _accounts(s, seed, stream, norm):
    """The state of a layer that has run for a while: counts of some
    thousands, mean routing weights around 1 / E, C_s within a few percent
    of the experts' usual output norm."""
    g = _gen(seed, stream)
    n = torch.randint(1000, 4000, (s.E,), device=DEV, generator=g)
    share = torch.rand(s.E, device=DEV, generator=g) * 1.5 / s.E + 0.5 / s.E
    c = norm * (1.0 + 0.02 * torch.randn(s.E, device=DEV, generator=g))
    return n, (n * share).float(), c.float()


# output norm of a random SwiGLU expert over sqrt(d): inputs of variance 3
# (the clustered hidden states) or 1 (after a RMSNorm)
_NORM_X, _NORM_U = 1.75, 0.6


def _params(s, mode, packed, share):
    dt = L.EAT_BF16 if s.bf16 else L.EAT_F32
    return L.eat_params_default(mode=mode, E=s.E, d_model=s.d, d_ffn=s.F, top_k=s.K, top_p=s.top_p or 0.6,
                                inv_temperature=s.inv_temp, cs_mode=1 if share else 0, act_dtype=dt, expert_dtype=dt,
                                d_shared=s.F_shared,
                                weight_layout=L.EAT_LAYOUT_PACKED if packed else L.EAT_LAYOUT_ROWS)


def _layer_inputs(case, seed):
    s, T = SHAPES[case["shape"]], case["tokens"]
    x = _hidden(s, T, seed, 1)
    trend = None
    if case["trend"]:
        trend = torch.randint(-1, 2, (T,), device=DEV, generator=_gen(seed, 3)).to(torch.int8)
    return s, _weights(s, seed, 0), x, trend, _accounts(s, seed, 2, _NORM_X * math.sqrt(s.d))


def _stack_inputs(case, seed):
    s, n = SHAPES["stack16"], case["layers"]
    ws = [_weights(s, seed, 10 + 4 * l) for l in range(n)]
    mixes = [_normal(_gen(seed, 11 + 4 * l), (s.d, s.d), s.d ** -0.5, torch.bfloat16) for l in range(n)]
    accs = [_accounts(s, seed, 12 + 4 * l, _NORM_U * math.sqrt(s.d)) for l in range(n)]
    return s, ws, mixes, accs, _hidden(s, case["tokens"], seed, 1)


def _ppl_inputs(case, seed):
    S, d, V = case["sequences"], case["d"], case["vocab"]
    g = _gen(seed, 0)
    head = _normal(g, (V, d), d ** -0.5, torch.bfloat16)
    # two tokens per sequence, fed in turn
    return head, [(_normal(g, (S, d), 1.0, torch.bfloat16),
                   torch.randint(0, V, (S,), device=DEV, generator=g).to(torch.int32)) for _ in range(2)]


def prepare(case, seed):
    """The objects a program holds before the call: layers with their
    weights, workspace and accounts, and the call's inputs."""
    if case["kind"] == "ppl":
        head, tokens = _ppl_inputs(case, seed)
        return {"kind": "ppl", "signal": PplSignal(case["sequences"], head), "tokens": tokens, "at": 0}
    if case["kind"] == "stack":
        s, ws, mixes, accs, x = _stack_inputs(case, seed)
        if case["packed"]:
            ws = [pack_weights(w) for w in ws]
        params = [_params(s, case["mode"], case["packed"], False) for _ in ws]
        stack = EatStack(params, case["tokens"], ws, mixes)
        for lay, a in zip(stack.layers, accs):
            lay.load_accounts(*a)
        masks = torch.empty(case["layers"], case["tokens"], dtype=torch.int64, device=DEV)
        return {"kind": "stack", "stack": stack, "x": x, "masks": masks}
    s, w, x, trend, acc = _layer_inputs(case, seed)
    if case["packed"]:
        w = pack_weights(w)
    lay = EatLayer(_params(s, case["mode"], case["packed"], case["share"]), case["tokens"], w)
    lay.load_accounts(*acc)
    lay.workspace(case["tokens"])
    return {"kind": "layer", "layer": lay, "x": x, "trend": trend, "mask": lay.mask_tensor(case["tokens"]),
            "load": torch.empty(s.E, dtype=torch.int32, device=DEV)}


def run(state):
    if state["kind"] == "ppl":
        sig = state["signal"]
        h, target = state["tokens"][state["at"]]
        state["at"] ^= 1
        trend = sig.step(h, target)
        return {"trend": trend, "nll": sig.nll, "nll_sum": sig.nll_sum, "count": sig.count, "ppl": sig.ppl_prev}
    if state["kind"] == "stack":
        st = state["stack"]
        h = st.forward(state["x"], masks_out=state["masks"], rms_eps=EPS)
        return {"h": h, "masks": state["masks"], "n": [l.n for l in st.layers],
                "p_total": [l.p_total for l in st.layers], "c_s": [l.c_s for l in st.layers]}
    lay = state["layer"]
    y = lay.forward(state["x"], state["trend"], mask_out=state["mask"], load_out=state["load"])
    return {"y": y, "mask": state["mask"], "load": state["load"], "n": lay.n, "p_total": lay.p_total, "c_s": lay.c_s}


# -------------------------------------------------------------------- work --

def _layer_work(s, T, mode):
    """Bytes and flops of one layer: the weights of the experts in use, the
    router, x and y once; the selected rows' products."""
    k = TOPP_K[s.name] if mode == "topp" else s.K
    used = min(s.E, k) if mode == "eat" else s.E * (1.0 - (1.0 - k / s.E) ** T)
    es = 2 if s.bf16 else 4
    nbytes = (3.0 * s.d * s.F * used + 3.0 * s.d * s.F_shared) * es + 4.0 * s.E * s.d + 2.0 * T * s.d * es
    flops = 6.0 * T * k * s.d * s.F + 6.0 * T * s.d * s.F_shared + 2.0 * T * s.d * s.E
    return nbytes, flops


def work(case):
    if case["kind"] == "ppl":
        S, d, V = case["sequences"], case["d"], case["vocab"]
        return {"bytes": 2.0 * d * V + 2.0 * S * d, "flops": 2.0 * S * d * V}
    if case["kind"] == "stack":
        s, n, T = SHAPES["finegrained"], case["layers"], case["tokens"]
        b, f = _layer_work(s, T, case["mode"])
        return {"bytes": n * (b + 2.0 * s.d * s.d), "flops": n * (f + 2.0 * T * s.d * s.d)}
    # the share reading keeps every expert in use, like Top-K
    mode = "topk" if case["mode"] == "eat" and case["share"] else case["mode"]
    b, f = _layer_work(SHAPES[case["shape"]], case["tokens"], mode)
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Largest difference two correct implementations show (about four times
    what a comparison with ``exact`` shows): fp32 sums in another order; one
    bf16 rounding of the hidden rows and of y (and of the expert rows in
    large calls); several in stacked layers.  ``differ``: a routing decision
    on a tie of the 32-bit router scores."""
    if case["kind"] == "ppl":
        return {"rel": 1e-5, "differ": 0.005}
    if case["kind"] == "stack":
        return {"rel": 0.03, "differ": 0.005}
    if not SHAPES[case["shape"]].bf16:
        return {"rel": 1e-5, "differ": 0.002}
    return {"rel": 0.012, "differ": 0.002}


# ------------------------------------------------------------------- exact --

def _route64(s, x, w_router, mode, share, trend, acc):
    """Routing in 64 bits: the probabilities, the selection and the gates."""
    p = torch.softmax(x.double() @ w_router.double().T * s.inv_temp, dim=1)
    T, E = p.shape
    if mode == "topk":
        m = torch.zeros_like(p, dtype=torch.bool).scatter_(1, p.topk(s.K, dim=1).indices, True)
    elif mode == "topp":
        v, order = torch.sort(p, dim=1, descending=True, stable=True)
        before = torch.cumsum(v, dim=1) - v
        m = torch.zeros_like(p, dtype=torch.bool).scatter_(1, order, before < (s.top_p or 0.6))
    else:
        n, pt, c = (a.double() for a in acc)
        hist = 0.3 * n / n.sum() + 0.3 * torch.where(n > 0, pt / n.clamp(min=1), 0.0) + 0.4 * (c / c.sum() if share else c)
        imp = 0.4 * p + 0.6 * hist
        mu, sd = p.mean(dim=1), p.std(dim=1, correction=0)
        tau = torch.maximum(0.5 * mu, mu - sd)
        up = (trend > 0) if trend is not None else torch.zeros(T, dtype=torch.bool, device=p.device)
        tau = 0.7 * torch.where(up, 1.2, 0.9) * tau + 0.3 * tau
        v = torch.sort(p, dim=1).values

        def point(q):
            h = q * (E - 1)
            lo = int(math.floor(h))
            return v[:, lo] + (h - lo) * (v[:, min(lo + 1, E - 1)] - v[:, lo])

        tau = torch.minimum(torch.maximum(tau, point(0.1)), point(0.9))
        cand = imp > tau[:, None]
        val = torch.where(cand, imp, -math.inf)
        kth = val.topk(s.K, dim=1).values[:, -1:]
        m = cand & (val >= kth)
        none = ~cand.any(dim=1)
        m[none] = torch.nn.functional.one_hot(imp.argmax(dim=1), E).bool()[none]
    g = p * m
    return p, m, g / (g.sum(dim=1, keepdim=True) + 1e-8)


def _swiglu64(x, w1, w3, w2):
    a = x.double()
    return (torch.nn.functional.silu(a @ w1.double().T) * (a @ w3.double().T)) @ w2.double().T


def _layer64(s, w, x, mode, share, trend, acc):
    """(y, new P_total, new C_s) of one layer in 64 bits."""
    p, m, g = _route64(s, x, w["w_router"], mode, share, trend, acc)
    y = torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    n, pt, c = acc
    pt, c = pt.double().clone(), c.double().clone()
    for e in range(s.E):
        rows = m[:, e].nonzero()[:, 0]
        if rows.numel() == 0:
            continue
        o = _swiglu64(x[rows], w["w1"][e], w["w3"][e], w["w2"][e])
        y.index_add_(0, rows, g[rows, e, None] * o)
        if mode == "eat":
            pt[e] += p[rows, e].sum()
            c[e] = 0.05 * c[e] + 0.95 * o.norm(dim=1).mean()
    if s.F_shared:
        y += _swiglu64(x, w["ws1"], w["ws3"], w["ws2"])
    return y, pt, c


def exact(case, seed):
    if case["kind"] == "ppl":
        head, ((h, target), _) = _ppl_inputs(case, seed)
        z = h.double() @ head.double().T
        nll = torch.logsumexp(z, dim=1) - z.gather(1, target.long()[:, None])[:, 0]
        return {"trend": None, "nll": nll, "nll_sum": nll, "count": None, "ppl": torch.exp(nll)}
    if case["kind"] == "stack":
        s, ws, mixes, accs, x = _stack_inputs(case, seed)
        # the bf16 roundings between the layers are part of what the stack computes
        h, pts, cs = x.double(), [], []
        for w, mix, acc in zip(ws, mixes, accs):
            u = (h / torch.sqrt((h * h).mean(dim=1, keepdim=True) + EPS)).to(torch.bfloat16)
            y, pt, c = _layer64(s, w, u, case["mode"], False, None, acc)
            r = (h + y).to(torch.bfloat16).double()
            h = (r @ mix.double().T).to(torch.bfloat16).double()
            pts.append(pt)
            cs.append(c)
        return {"h": h, "masks": None, "n": [None] * len(ws), "p_total": pts, "c_s": cs}
    s, w, x, trend, acc = _layer_inputs(case, seed)
    y, pt, c = _layer64(s, w, x, case["mode"], case["share"], trend, acc)
    return {"y": y, "mask": None, "load": None, "n": None, "p_total": pt, "c_s": c}
