"""The work a user has this framework do, as measurable cases.

Every case goes through the public entry points: the fused layer (``MoELayer.forward``),
the stage entry points of the C ABI, and the decoding loop (``run_trajectory``).  Shapes are
the repository's own: the tiny test layer, the LLaDA-MoE layer (d 2048, 64 experts of width
1024) and the LLaDA2.0-mini layer (d 2048, 256 experts of width 512, one shared expert), over
1 to 16384 tokens.  A case's tokens are either whole sequences (prompt and all target blocks,
as the paper runs them) or only the active 32-token block of each sequence, the call that a
block-cached decoder makes.

Inputs follow ``synth``: h ~ N(0, 1), weights ~ N(0, 0.02), confidences Beta(2, 2) with steps
U(-0.2, 0.3), hyper-parameters of the paper's Section 5.1.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import torch

from paper_2608_01784_amd import _lib
from paper_2608_01784_amd.layer import ExpertWeights, MoELayer, TokenState
from paper_2608_01784_amd.trajectory import run_trajectory

THETA = 0.9
BLOCK = 32          # tokens per target block
RULES = {"budget": 0, "uniform": 0, "topp": 1, "threshold": 2}

# d, experts, expert width, shared width; K_base, delta_role, delta_cur, K_min, K_max, w_cf
MODELS = {
    "tiny": (256, 8, 512, 0, 2, 1, 1, 1, 4, 0.30),
    "llada": (2048, 64, 1024, 0, 8, 4, 2, 2, 12, 0.30),
    "mini": (2048, 256, 512, 512, 8, 4, 2, 2, 12, 0.25),
    "skewed": (2048, 256, 512, 0, 8, 4, 2, 1, 16, 0.30),
}


def listed():
    return [
        # fixed top-8 over the last few open positions of a generation: the smallest call
        dict(name="tail_llada_t5", kind="layer", model="llada", T=5, seq=5, counts="uniform",
             layers=1, norm=1, thr=0.0),
        # the layer of the test suite and of smoke(): launches and latency
        dict(name="tiny_t128", kind="layer", model="tiny", T=128, seq=128, counts="budget",
             layers=1, norm=1, thr=0.0),
        # one active block of one sequence, its prompt and past blocks cached
        dict(name="block_llada_t32", kind="layer", model="llada", T=32, seq=32, counts="budget",
             layers=1, norm=1, thr=0.0),
        # the active blocks of three sequences, 256 experts and the shared expert
        dict(name="blocks_mini_t96", kind="layer", model="mini", T=96, seq=32, counts="budget",
             layers=1, norm=1, thr=0.0),
        # score-derived counts over the full softmax, an odd number of tokens
        dict(name="topp_mini_t777", kind="layer", model="mini", T=777, seq=259, counts="topp",
             layers=1, norm=0, thr=0.15),
        # one whole sequence (512 prompt tokens, 16 blocks)
        dict(name="seq_llada_t1024", kind="layer", model="llada", T=1024, seq=1024,
             counts="budget", layers=1, norm=1, thr=0.0),
        # the six stage entry points one by one, ragged sequences
        dict(name="stages_llada_t2731", kind="stages", model="llada", T=2731, seq=911,
             counts="budget", layers=1, norm=1, thr=0.0),
        # the fixed-count baseline of the paper (default token-choice routing)
        dict(name="uniform_llada_t3000", kind="layer", model="llada", T=3000, seq=1024,
             counts="uniform", layers=1, norm=0, thr=0.0),
        # a batch of four sequences, 256 experts and the shared expert
        dict(name="batch_mini_t4096", kind="layer", model="mini", T=4096, seq=1024,
             counts="budget", layers=1, norm=1, thr=0.0),
        # decoding: eight denoising forwards with the state update between them
        dict(name="decode_llada_t1024", kind="decode", model="llada", T=1024, seq=1024,
             counts="budget", layers=1, norm=1, thr=0.0),
        # the largest layer: 256 short sequences, Zipf-skewed experts
        dict(name="skewed_t16384", kind="layer", model="skewed", T=16384, seq=64,
             counts="budget", layers=1, norm=1, thr=0.0),
        # a whole call: four stacked layers that share one count vector, with residuals
        dict(name="stack_llada_t8192", kind="layer", model="llada", T=8192, seq=1024,
             counts="budget", layers=4, norm=1, thr=0.0),
    ]


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["stages"] * 2 + ["decode"])
    model = rng.choice(["llada", "llada", "llada", "mini", "mini", "skewed", "tiny"])
    top = {"layer": 16384, "stages": 16384, "decode": 1024}[kind]
    T = max(1, min(top, int(round(2.0 ** rng.uniform(0.0, np.log2(top))))))
    if rng.random() < 0.25:      # the round sizes are as common as the odd ones
        T = min(top, max(1, 32 * ((T + 31) // 32)))
    seq = rng.choice([32, 64, 259, 1024]) if T > 32 else T
    counts = "budget" if kind == "decode" else rng.choice(["budget"] * 4 + ["uniform", "topp", "threshold"])
    thr = {"topp": rng.choice([0.15, 0.25, 0.325]), "threshold": rng.choice([0.0190, 0.0270])}.get(counts, 0.0)
    layers = 2 if kind == "layer" and T <= 4096 and rng.random() < 0.2 else 1
    return dict(kind=kind, model=model, T=T, seq=min(seq, T), counts=counts, layers=layers,
                norm=rng.choice([1, 1, 0]), thr=thr)


# ---- inputs -------------------------------------------------------------------------------
@dataclasses.dataclass(frozen=True)
class Params:
    k_base: int
    delta_role: int
    delta_cur: int
    k_min: int
    k_max: int
    q: float
    theta: float
    w_cf: float
    v_ref: float
    tau: float
    signal: int = 0


def _params(case):
    kb, dr, dc, lo, hi, w_cf = MODELS[case["model"]][4:]
    return Params(kb, dr, dc, lo, hi, 0.25, THETA, w_cf, 0.01, 0.05)


def _tokens(case, seed, fresh):
    """Token state as numpy arrays.  fresh: the start of a generation (all targets masked,
    block 1 active, no confidence history)."""
    rng = np.random.default_rng([seed, 9])
    T, seq = case["T"], case["seq"]
    block, masked, offs, active = [], [], [0], []
    while offs[-1] < T:
        n = min(seq, T - offs[-1])
        if seq <= BLOCK:                       # the active block alone
            a, b = 1 + int(rng.integers(16)), None
            b = np.full(n, a, np.int32)
            first = 0
        else:
            n_prompt = (seq // 2) // BLOCK * BLOCK
            n_blocks = -(-(seq - n_prompt) // BLOCK)
            a = 1 if fresh else 1 + int(rng.integers(n_blocks))
            b = np.concatenate([np.zeros(n_prompt, np.int32),
                                1 + np.arange(seq - n_prompt, dtype=np.int32) // BLOCK])[:n]
            first = n_prompt
        m = (b > (0 if fresh else a)).astype(np.uint8)
        if seq <= BLOCK:
            m[:] = 1 if fresh else 0
        if not fresh:
            own = np.flatnonzero(b == a)
            if len(own):
                n_open = min(len(own), max(1, int(round(float(rng.uniform(0.2, 0.9)) * len(own)))))
                m[rng.choice(own, size=n_open, replace=False)] = 1
        m[:first] = 0
        block.append(b)
        masked.append(m)
        active.append(a)
        offs.append(offs[-1] + n)
    c1 = rng.beta(2.0, 2.0, T).astype(np.float32)
    c2 = np.clip(c1 - rng.uniform(-0.2, 0.3, T).astype(np.float32), 0, 1).astype(np.float32)
    m = np.concatenate(masked)
    hist = np.where(m == 1, 2, 0).astype(np.int8)
    if fresh:
        c1, c2, hist = np.zeros_like(c1), np.zeros_like(c2), np.zeros_like(hist)
    return dict(block_idx=np.concatenate(block).astype(np.int32), masked=m, hist_len=hist,
                conf_prev1=c1, conf_prev2=c2, seq_offsets=np.array(offs, np.int32),
                active_block=np.array(active, np.int32))


FORWARDS = 8


def _confidence(case, seed):
    rng = np.random.default_rng([seed, 21])
    T = case["T"]
    base, rate = rng.beta(2.0, 5.0, T), rng.uniform(0.03, 0.2, T)
    t = np.arange(FORWARDS)[:, None]
    return np.clip(base + rate * t + rng.normal(0.0, 0.02, (FORWARDS, T)), 0, 1).astype(np.float32)


def _tensors(case, seed):
    """h, the layers' weights and the residual rows, on the GPU."""
    d, E, f, fs = MODELS[case["model"]][:4]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 17)

    def normal(*shape, scale=1.0, dtype=torch.bfloat16):
        x = torch.empty(shape, dtype=dtype, device="cuda")
        return x.normal_(0.0, scale, generator=g)

    bias = None
    if case["model"] == "skewed":
        perm = np.random.default_rng([seed, 12]).permutation(E) + 1.0
        bias = torch.from_numpy((-1.2 * np.log(perm)).astype(np.float32)).cuda()
    weights = []
    for _ in range(case["layers"]):
        w = dict(w_gate=normal(E, f, d, scale=0.02), w_up=normal(E, f, d, scale=0.02),
                 w_down=normal(E, d, f, scale=0.02),
                 w_router=normal(E, d, scale=0.02, dtype=torch.float32), router_bias=bias)
        if fs:
            w.update(ws_gate=normal(fs, d, scale=0.02), ws_up=normal(fs, d, scale=0.02),
                     ws_down=normal(d, fs, scale=0.02))
        weights.append(ExpertWeights(**w))
    h = normal(case["T"], d)
    rho = [normal(case["T"], d, scale=0.1) for _ in range(case["layers"])] if case["layers"] > 1 else []
    return h, weights, rho


def _uniform(case):
    return MODELS[case["model"]][4] if case["counts"] == "uniform" else 0


def prepare(case, seed):
    fresh = case["kind"] == "decode"
    tok = _tokens(case, seed, fresh)
    h, weights, rho = _tensors(case, seed)
    prm = _params(case)
    state = {n: torch.from_numpy(v).cuda() for n, v in tok.items()}
    s = dict(case=case, h=h, weights=weights, rho=rho, prm=prm, state=state)
    if case["kind"] == "stages":
        T, w = case["T"], weights[0]
        d, E, f = h.shape[1], w.E, w.f
        kcap = _uniform(case) or prm.k_max
        cap = T * kcap

        def i32(n):
            return torch.zeros(n, dtype=torch.int32, device="cuda")

        s.update(kcap=kcap, logits=torch.zeros(T, E, device="cuda"), k=i32(T), pairs=i32(1),
                 off=i32(T + 1), pexp=i32(cap), pw=torch.zeros(cap, device="cuda"), eo=i32(E + 1),
                 tok=i32(cap), pos=i32(cap),
                 pws=torch.zeros(max(256, _lib.reflex_permute_workspace_size(cap, E)),
                                 dtype=torch.uint8, device="cuda"),
                 gws=torch.zeros(max(256, _lib.reflex_swiglu_workspace_size(cap, E, f)),
                                 dtype=torch.uint8, device="cuda"),
                 y=torch.empty(cap, d, dtype=torch.bfloat16, device="cuda"),
                 out=torch.empty(T, d, dtype=torch.bfloat16, device="cuda"))
        if case["counts"] == "uniform":
            s["k"].fill_(kcap)
            s["pairs"].fill_(cap)
        return s
    s["layers"] = [MoELayer(case["T"], h.shape[1], w, prm, uniform_k=_uniform(case),
                            norm_topk=case["norm"], k_rule=RULES[case["counts"]],
                            k_threshold=case["thr"]) for w in weights]
    if fresh:
        s["conf"] = torch.from_numpy(_confidence(case, seed)).cuda()
    return s


# ---- one pass -----------------------------------------------------------------------------
def _run_stages(s):
    case, w, st, prm = s["case"], s["weights"][0], s["state"], s["prm"]
    _lib.reflex_router_logits(s["h"], w.w_router, w.router_bias, s["logits"])
    if case["counts"] == "budget":
        _lib.reflex_assign_budget(st["block_idx"], st["masked"], st["hist_len"], st["conf_prev1"],
                                  st["conf_prev2"], st["seq_offsets"], st["active_block"], prm,
                                  s["k"], s["pairs"])
    elif case["counts"] != "uniform":
        _lib.reflex_count_rule(s["logits"], RULES[case["counts"]], case["thr"], prm.k_min, prm.k_max,
                               s["k"], s["pairs"])
    _lib.reflex_topk_variable(s["logits"], s["k"], s["kcap"], case["norm"], s["off"], s["pexp"], s["pw"])
    _lib.reflex_permute(s["off"], s["pexp"], s["pairs"], w.E, s["eo"], s["tok"], s["pos"], s["pws"])
    _lib.reflex_grouped_swiglu(s["h"], s["tok"], s["eo"], w.w_gate, w.w_up, w.w_down, s["y"], s["gws"])
    _lib.reflex_combine(s["y"], s["off"], s["pos"], s["pw"], None, s["out"])
    return {"out": s["out"], "logits": s["logits"], "k": s["k"], "offsets": s["off"],
            "pairs": s["pairs"]}


def run(s):
    case = s["case"]
    if case["kind"] == "stages":
        return _run_stages(s)
    layers = s["layers"]
    if case["kind"] == "decode":
        # a generation begins from the prompt's state, which the loop then advances in place
        st = TokenState(**{n: v.clone() for n, v in s["state"].items()})
        conf = s["conf"]
        stats = run_trajectory(layers[0], s["h"], st, lambda t: conf[t], THETA, min_commit=1,
                               max_forwards=FORWARDS)
        return {"out": layers[0].out, "logits": layers[0].logits, "k": layers[0].k,
                "masked": st.masked, "hist": st.hist_len, "conf1": st.conf_prev1,
                "conf2": st.conf_prev2, "active": st.active_block,
                "pairs": [int(p) for p in stats.pairs]}
    st = TokenState(**s["state"])
    if len(layers) == 1:
        out = layers[0].forward(s["h"], st)
    else:
        x, k = s["h"], None
        for lay, rho in zip(layers, s["rho"]):
            x = lay.forward(x, st, k_in=k, residual_a=x, residual_b=rho)
            k = lay.k if k is None else k
        out = x
    return {"out": out, "logits": [lay.logits for lay in layers], "k": layers[0].k,
            "pairs": [lay.pairs for lay in layers]}


# ---- what a pass cannot do without ----------------------------------------------------------
# mean count of each score rule on softmax masses of N(0, 0.9) scores (tiny: N(0, 0.32)) by the
# number of experts, before the bounds
RULE_COUNTS = {("topp", 0.15): {8: 1.0, 64: 2.5, 256: 7.5}, ("topp", 0.25): {8: 2.0, 64: 4.6, 256: 15.5},
               ("topp", 0.325): {8: 2.3, 64: 6.5, 256: 23.2},
               ("threshold", 0.0190): {8: 8, 64: 16.4, 256: 3.5},
               ("threshold", 0.0270): {8: 8, 64: 9.5, 256: 1.2}}


def _avg_k(case):
    E = MODELS[case["model"]][1]
    kb, dr, _, lo, hi = MODELS[case["model"]][4:9]
    if case["counts"] == "uniform":
        return kb
    if case["counts"] in ("topp", "threshold"):
        return min(hi, max(lo, RULE_COUNTS[case["counts"], case["thr"]][E]))
    if case["kind"] == "decode":
        return 0.75 * (kb + dr)                       # the first blocks: most tokens are prompt
    return min(hi, kb + dr) if case["seq"] <= 64 else 5 if case["model"] != "tiny" else 2


def work(case):
    d, E, f, fs = MODELS[case["model"]][:4]
    T, n = case["T"], case["layers"] * (FORWARDS if case["kind"] == "decode" else 1)
    P = T * _avg_k(case)
    # experts that some token chooses, the pairs falling on them evenly or (skewed) by rank^-1.2
    share = np.arange(1, E + 1.0) ** (-1.2 if case["model"] == "skewed" else 0.0)
    touched = float(np.sum(1.0 - (1.0 - share / share.sum()) ** P))
    row = T * d * 2
    own = 2 + (2 if case["layers"] > 1 else 0)       # h read, out written, residuals read
    return {"bytes": n * (touched * 3 * f * d * 2 + 3 * fs * d * 2 + own * row + E * d * 4 + T * E * 4),
            "flops": n * (6.0 * d * f * P + 6.0 * d * fs * T + 2.0 * T * E * d)}


def tolerance(case):
    # The activation, the expert rows and the output are each rounded to bf16 once: 3e-3 against
    # 64 bits.  `max` is wide because two scores of one token that agree to the last bits of fp32
    # may change places where the sums run in another order, and that token then has another
    # expert.  Counts are whole numbers decided in fp64: a count may differ only where a rule's
    # mass lies on its threshold to fp32 rounding of the scores.  From layer to layer of a stack a
    # bf16 rounding of the hidden rows moves near ties of the next router: four layers are up to
    # 0.015 off the 64-bit result, twice that apart from each other.
    return {"rel": 1e-2 if case["layers"] == 1 else 0.03, "max": 0.99, "differ": 0.0 if case["counts"] in ("budget", "uniform") else 2e-3}


# ---- the same in 64 bits -------------------------------------------------------------------
def _logistic(x):
    return 1.0 / (1.0 + np.exp(-x))


def _budget(tok, p):
    """Counts of Eqs. (5)-(9), one sequence at a time."""
    f64 = lambda v: float(np.float32(v))      # noqa: E731  (parameters are stored as float32)
    q, theta, w, v_ref, tau = (f64(v) for v in (p.q, p.theta, p.w_cf, p.v_ref, p.tau))
    k = np.zeros(len(tok["block_idx"]), np.int64)
    for s, a in enumerate(tok["active_block"]):
        lo, hi = tok["seq_offsets"][s], tok["seq_offsets"][s + 1]
        b, m, hl = tok["block_idx"][lo:hi], tok["masked"][lo:hi], tok["hist_len"][lo:hi]
        dist = np.abs(b.astype(np.int64) - int(a))
        ks = np.where(dist <= 1, p.k_base + p.delta_role,
                      np.where(dist == 2, p.k_base, p.k_base - p.delta_role))
        j = np.flatnonzero((m != 0) & (b == a) & (hl >= 1))
        if len(j):
            c1 = tok["conf_prev1"][lo:hi][j].astype(np.float64)
            c2 = tok["conf_prev2"][lo:hi][j].astype(np.float64)
            two = hl[j] >= 2
            v = np.where(two, np.clip(c1 - c2, -w / 2, w / 2), 0.0)
            c = np.where(two, np.clip(c1 + v, 0.0, 1.0), c1)
            F = _logistic((c - theta + w) / tau) * _logistic((theta - c) / tau)
            S = F * np.where(two, _logistic((v_ref - v) / tau), 1.0)
            order = j[np.lexsort((j, -S))]
            n_q = int(np.floor(q * len(j)))
            cur = p.k_base + p.delta_role
            ks[order[:n_q]] = cur + p.delta_cur
            ks[order[len(j) - n_q:]] = cur - p.delta_cur
        k[lo:hi] = np.clip(ks, p.k_min, p.k_max)
    return k


def _advance(tok, conf):
    """Eq. (1) with the progress guard, in place."""
    for s in range(len(tok["active_block"])):
        lo, hi = tok["seq_offsets"][s], tok["seq_offsets"][s + 1]
        b, m, a = tok["block_idx"][lo:hi], tok["masked"][lo:hi], tok["active_block"][s]
        c = conf[lo:hi]
        own = np.flatnonzero((m != 0) & (b == a))
        commit = own[c[own] >= np.float32(THETA)]
        if len(own) and not len(commit):
            commit = own[[int(np.argmax(c[own]))]]
        was = m != 0
        tok["conf_prev2"][lo:hi][was] = tok["conf_prev1"][lo:hi][was]
        tok["conf_prev1"][lo:hi][was] = c[was]
        tok["hist_len"][lo:hi][was] = np.minimum(tok["hist_len"][lo:hi][was] + 1, 2)
        m[commit] = 0
        if not np.any((m != 0) & (b == a)) and a < b.max():
            tok["active_block"][s] = a + 1


def _counts(case, prob, rank):
    """Top-p and Expert-Threshold counts from the routing mass."""
    if case["counts"] == "topp":
        cum = prob.gather(1, rank).cumsum(1)
        k = (cum < float(np.float32(case["thr"]))).sum(1) + 1
    else:
        k = (prob > float(np.float32(case["thr"]))).sum(1)
    lo, hi = MODELS[case["model"]][7:9]
    return k.clamp(lo, hi)


def _expert(x, wg, wu, wd):
    g, u = x @ wg.double().t(), x @ wu.double().t()
    return (g * torch.sigmoid(g) * u) @ wd.double().t()


def _layer(case, x, w, k):
    """One layer in float64; k: [T] counts or None for a score rule."""
    logits = x @ w.w_router.double().t()
    if w.router_bias is not None:
        logits = logits + w.router_bias.double()
    rank = torch.sort(logits, dim=1, descending=True, stable=True).indices
    prob = torch.softmax(logits, 1)
    if k is None:
        k = _counts(case, prob, rank)
    chosen = torch.arange(w.E, device="cuda")[None, :] < k[:, None]
    sel = torch.zeros_like(chosen).scatter_(1, rank, chosen)
    alpha = torch.where(sel, prob, torch.zeros_like(prob))
    if case["norm"]:
        alpha = alpha / alpha.sum(1, keepdim=True).clamp_min(1e-300)
    out = torch.zeros_like(x)
    for e in range(w.E):
        rows = sel[:, e].nonzero()[:, 0]
        if len(rows):
            y = _expert(x[rows], w.w_gate[e], w.w_up[e], w.w_down[e])
            out.index_add_(0, rows, alpha[rows, e][:, None] * y)
    if w.ws_gate is not None and case["kind"] != "stages":
        out += _expert(x, w.ws_gate, w.ws_up, w.ws_down)
    return out, logits, k


def exact(case, seed):
    fresh = case["kind"] == "decode"
    tok = _tokens(case, seed, fresh)
    h, weights, rho = _tensors(case, seed)
    prm = _params(case)
    pairs = []
    if fresh:
        conf = _confidence(case, seed)
        for t in range(FORWARDS):
            k = _budget(tok, prm)
            pairs.append(int(k.sum()))
            _advance(tok, conf[t])
            if not tok["masked"].any():
                break
    elif case["counts"] == "budget":
        k = _budget(tok, prm)
    elif case["counts"] == "uniform":
        k = np.full(case["T"], prm.k_base)
    else:
        k = None
    k = None if k is None else torch.from_numpy(np.asarray(k)).cuda()
    x, logits = h.double(), []
    for i, w in enumerate(weights):
        out, r, k = _layer(case, x, w, k)
        logits.append(r)
        x = out if not rho else x + out + rho[i].double()
    k32 = k.to(torch.int32)
    total = k32.sum().reshape(1).to(torch.int32)
    if case["kind"] == "stages":
        off = torch.cat([torch.zeros(1, dtype=torch.int32, device="cuda"), k32.cumsum(0).to(torch.int32)])
        return {"out": x, "logits": logits[0], "k": k32, "offsets": off, "pairs": total}
    if fresh:
        dev = {n: torch.from_numpy(tok[n]).cuda() for n in ("masked", "hist_len", "conf_prev1", "conf_prev2", "active_block")}
        return {"out": x, "logits": logits[0], "k": k32, "masked": dev["masked"], "hist": dev["hist_len"],
                "conf1": dev["conf_prev1"], "conf2": dev["conf_prev2"], "active": dev["active_block"],
                "pairs": pairs}
    return {"out": x, "logits": logits, "k": k32, "pairs": [total] * len(weights)}
