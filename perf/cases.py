"""Measured workloads of the sparse dReLU FFN / MoE decode path.

A case is one decode step's FFN (or MoE) work: `layers` independent layers of
one shape, each called once through the public binding with the weights, the
workspace and the output buffer that a serving program keeps.  Layer shapes
are the repository's own (Mistral-7B FFN: hidden 4096, inter 14336; Mixtral:
8 experts of that shape, top 2; the small fp32 layer 512 x 1792) or generic.
Weights are drawn as in the repository's synthetic recipe: N(0, 1/hidden),
x ~ N(0, 1) with x[:, 0] = 1 and the gate's column 0 set to a bias b, so that
an open gate has probability p_gate = Phi(b).

`layers` is chosen so that a pass streams its weights from HBM (several
hundred MB per pass) as the steps of a whole model do.
"""
import math
from statistics import NormalDist

import torch

from paper_2406_05955_amd import binding as ts

DEV = "cuda"
F32, BF16 = "f32", "bf16"


def _case(entry, dtype, batch, hidden, inter, layers, p_gate, **more):
    c = {"entry": entry, "dtype": dtype, "batch": batch, "hidden": hidden, "inter": inter, "layers": layers,
         "p_gate": p_gate, "experts": 0, "top_k": 0, "tau": 0.0, "keep": 0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: the small fp32 layer, one token (latency and launches)
        _case("ffn", F32, 1, 512, 1792, 1, 0.2, name="ffn_f32_small_b1"),
        # the headline: one token through Mistral-shaped layers, 90% of Combined zero
        _case("ffn", BF16, 1, 4096, 14336, 4, 0.2, name="ffn_mistral_b1"),
        # small and ordinary decode batches
        _case("ffn", BF16, 8, 4096, 14336, 4, 0.2, name="ffn_mistral_b8"),
        _case("ffn", BF16, 32, 4096, 14336, 4, 0.2, name="ffn_mistral_b32"),
        # the largest batch the interface takes (a large decode batch, or a slice of a prompt)
        _case("ffn", BF16, 256, 4096, 14336, 2, 0.2, name="ffn_mistral_b256"),
        # fp32 weights with several tokens, ragged sizes
        _case("ffn", F32, 6, 2052, 5003, 4, 0.2, name="ffn_f32_ragged_b6"),
        # Mixtral-shaped MoE: one token, a decode batch, a large decode batch (97% zero inside an expert)
        _case("moe", BF16, 1, 4096, 14336, 1, 0.06, experts=8, top_k=2, name="moe_mixtral_b1"),
        _case("moe", BF16, 16, 4096, 14336, 1, 0.06, experts=8, top_k=2, name="moe_mixtral_b16"),
        _case("moe", BF16, 128, 4096, 14336, 1, 0.06, experts=8, top_k=2, name="moe_mixtral_b128"),
        # an activation predictor's neuron lists, one token
        _case("given", BF16, 1, 4096, 14336, 4, 0.2, name="given_mistral_b1"),
        # the shifted gate-only ReLU (10% open gates), a small decode batch
        _case("act", BF16, 4, 4096, 14336, 4, 0.2, tau=0.44, name="act_mistral_b4"),
        # the top-k magnitude mask at 95% sparsity, one token
        _case("topk", BF16, 1, 4096, 14336, 4, 0.2, keep=716, name="topk_mistral_b1"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: every entry point, both weight types,
    batches 1..256 and odd and ragged sizes."""
    entry = rng.choice(["ffn", "ffn", "ffn", "moe", "moe", "given", "act", "topk"])
    dtype = F32 if rng.random() < 0.25 else BF16
    step = 4 if dtype == F32 else 8
    hidden = max(step, _log(rng, 512, 4096) // step * step)
    if entry == "given" and dtype == F32:
        hidden = min(hidden, 2048)
    inter = _log(rng, 1792, 14336)
    batch = _log(rng, 1, 256) if entry in ("ffn", "moe") else _log(rng, 1, 16)
    if dtype == F32:
        batch = min(batch, 32)
    p_gate = rng.choice([0.06, 0.1, 0.2, 0.3, 0.5])
    layers = rng.choice([1, 2, 4])
    if entry == "moe":
        experts = rng.choice([4, 8, 16])
        if dtype == F32:
            experts, inter = 4, min(inter, 6000)
        return _case(entry, dtype, min(batch, 128), hidden, inter, 1, p_gate, experts=experts, top_k=rng.choice([1, 2]))
    if entry == "act":
        return _case(entry, dtype, batch, hidden, inter, layers, p_gate, tau=rng.choice([0.0, 0.25, 0.44]))
    if entry == "topk":
        return _case(entry, dtype, batch, hidden, inter, layers, p_gate, keep=max(1, int(inter * rng.choice([0.02, 0.05, 0.1]))))
    return _case(entry, dtype, batch, hidden, inter, layers, p_gate)


# ---------------------------------------------------------------------------

def _inputs(case, seed, layer):
    """The tensors of one layer on the GPU, from the seed alone."""
    B, H, I, E = case["batch"], case["hidden"], case["inter"], case["experts"]
    td = torch.float32 if case["dtype"] == F32 else torch.bfloat16
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + layer)
    s = 1.0 / math.sqrt(H)

    def randn(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)

    bias = NormalDist().inv_cdf(case["p_gate"])
    d = {"x": randn(B, H)}
    d["x"][:, 0] = 1.0
    lead = (E,) if E else ()
    if E:
        d["w_router"] = (randn(E, H) * s).to(td)
    for name in ("w_gate", "w_up", "w_down_t"):
        w = torch.empty(*lead, I, H, device=DEV, dtype=td)
        for e in range(max(E, 1)):
            m = randn(I, H).mul_(s)
            if name == "w_gate":
                m[:, 0] = bias
            (w[e] if E else w).copy_(m)
        d[name] = w
    if case["entry"] == "given":
        # the predictor: the gate's sign seen through noise, so the lists miss
        # a few open gates and hold some closed ones; a fixed capacity with
        # room above the expected length, ascending lists of differing lengths
        score = d["x"] @ d["w_gate"].float().T + 0.1 * randn(B, I)
        cap = min(I, int(1.25 * (case["p_gate"] + 0.01) * I) + 64)
        on = score > 0
        d["count"] = on.sum(dim=1).clamp(max=cap).to(torch.int32)
        order = torch.argsort((~on).to(torch.int8), dim=1, stable=True)[:, :cap]
        d["idx"] = order.to(torch.int32).contiguous()
    return d


def prepare(case, seed):
    B, H, I = case["batch"], case["hidden"], case["inter"]
    dt = ts.TS_F32 if case["dtype"] == F32 else ts.TS_BF16
    layers = [_inputs(case, seed, n) for n in range(case["layers"])]
    if case["entry"] == "moe":
        nb = ts.moe_workspace_bytes(B, H, I, case["experts"], case["top_k"], dt)
    elif case["entry"] == "given":
        nb = ts.ffn_given_workspace_bytes(B, H, I, layers[0]["idx"].shape[1], dt)
    else:
        nb = ts.ffn_workspace_bytes(B, H, I, dt)
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
    out = [torch.empty(B, H, dtype=torch.float32, device=DEV) for _ in layers]
    return {"case": case, "layers": layers, "ws": ws, "out": out}


def run(state):
    """One decode step: every layer once, in order, on the current stream."""
    c, ws = state["case"], state["ws"]
    entry, got = c["entry"], []
    for d, out in zip(state["layers"], state["out"]):
        w = (d["w_gate"], d["w_up"], d["w_down_t"])
        if entry == "ffn":
            got.append(ts.ffn_sparse(d["x"], *w, out=out, ws=ws))
        elif entry == "moe":
            got.append(ts.moe_sparse(d["x"], d["w_router"], *w, c["top_k"], out=out, ws=ws))
        elif entry == "given":
            got.append(ts.ffn_sparse_given(d["x"], *w, d["idx"], d["count"], out=out, ws=ws))
        elif entry == "act":
            got.append(ts.ffn_sparse_act(d["x"], *w, ts.TS_ACT_RELU_GATE, c["tau"], out=out, ws=ws))
        else:
            got.append(ts.ffn_sparse_topk(d["x"], *w, c["keep"], out=out, ws=ws))
    return got


def work(case):
    """Bytes and operations of one pass at the expected activity: W_gate once
    (for each expert that a token is routed to), the W_up / W_down rows that
    some token of the batch needs once, x and out once; two operations per
    weight element and token that needs it."""
    B, H, I, E, K = case["batch"], case["hidden"], case["inter"], case["experts"], case["top_k"]
    es = 4 if case["dtype"] == F32 else 2
    p = case["p_gate"]
    if case["entry"] == "act":
        p = NormalDist().cdf(NormalDist().inv_cdf(p) - case["tau"])
    pa = p if case["entry"] == "act" else p / 2
    if case["entry"] == "topk":
        pa = min(pa, case["keep"] / I)
    sets, tok = (E, B * K / E) if E else (1, B)  # weight sets, tokens of each on average

    def rows(q):
        """Expected rows that one weight set reads, each with probability q per token."""
        if not E:
            return I * (1 - (1 - q) ** B)
        return I * (1 - (1 - q * K / E) ** B)

    gate_rows = I * (1 - (1 - K / E) ** B) if E else I
    gate_tok = 1.0
    if case["entry"] == "given":
        gate_rows, gate_tok = rows(p), p
    nbytes = sets * (gate_rows + rows(p) + rows(pa)) * H * es + 2 * B * H * 4
    flops = 2.0 * sets * tok * I * H * (gate_tok + p + pa)
    if E:
        nbytes += E * H * es
        flops += 2.0 * B * E * H
    return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * flops}


def tolerance(case):
    """Single-token and fp32 calls: fp32 sums in another order (measured 2e-7
    to 1.2e-6 against 64 bits).  Batches of bf16 weights: x and Combined to 16
    significant bits (measured 4e-6 to 6e-6).  The mask and the routing
    choose by fp32 values: a near tie may fall to either side."""
    batched = case["entry"] in ("ffn", "moe") and case["dtype"] == BF16 and case["batch"] > 1
    t = {"rel": 2.5e-5 if batched else 5e-6}
    if case["entry"] == "moe":
        t["differ"] = 0.005
    return t


def _combined(case, d, x, wg, wu):
    g, u = x @ wg.T, x @ wu.T
    if case["entry"] == "act":
        return (g - case["tau"]).clamp(min=0) * u
    h = g.clamp(min=0) * u.clamp(min=0)
    if case["entry"] == "topk" and case["keep"] < h.shape[1]:
        order = torch.argsort(h, dim=1, descending=True, stable=True)[:, :case["keep"]]
        h = torch.zeros_like(h).scatter(1, order, h.gather(1, order))
    if case["entry"] == "given":
        cap = d["idx"].shape[1]
        on = torch.arange(cap, device=h.device)[None, :] < d["count"][:, None]
        m = torch.zeros_like(h).scatter(1, d["idx"].long(), on.to(h.dtype))
        h = h * m
    return h


def exact(case, seed):
    """The dense definition in 64-bit arithmetic."""
    outs = []
    for n in range(case["layers"]):
        d = _inputs(case, seed, n)
        x = d["x"].double()
        if case["entry"] != "moe":
            h = _combined(case, d, x, d["w_gate"].double(), d["w_up"].double())
            outs.append(h @ d["w_down_t"].double())
            continue
        K, E = case["top_k"], case["experts"]
        p = torch.softmax(x @ d["w_router"].double().T, dim=1)
        order = torch.argsort(p, dim=1, descending=True, stable=True)[:, :K]
        pw = p.gather(1, order)
        pw = pw / pw.sum(dim=1, keepdim=True)
        y = torch.zeros_like(x)
        for e in range(E):
            t, k = torch.nonzero(order == e, as_tuple=True)
            if t.numel():
                h = _combined(case, d, x[t], d["w_gate"][e].double(), d["w_up"][e].double())
                y.index_add_(0, t, (h @ d["w_down_t"][e].double()) * pw[t, k][:, None])
        outs.append((y, order.to(torch.int32), pw))
    return outs
