"""Performance cases of the SwiLA layer: what its users run, at the sizes of the
standard configurations and over the ranges around them.

Every case is one call of a public entry point on inputs that are already on the
GPU, with the outputs allocated by the call as a training or serving program
leaves it to do.  ``kind`` names the entry point:

  forward         forward             plain SwiLA over whole sequences
  temporal        forward_temporal    running priors (App. B.3)
  gated           forward_gated       per-key decay (App. B.4)
  gated_temporal  forward_gated       decay and running priors together
  backward        backward            gradients of the plain forward
  decode, decode_temporal, decode_gated, decode_gated_temporal
                                      one token per sequence, state in place

``dtype`` is that of the inputs and of o ("bf16" or "f32"); ``carry`` says that
the call starts from a state left by an earlier one (a later segment of a long
sequence, a chunked prefill) instead of zeros; ``recur`` draws the tokens from a
small vocabulary, so that keys come back as in retrieval-shaped text.

The App. D iteration (algo="newton") is not among the cases: it computes what
the exact forward computes, in ten to twenty sweeps that each cost more than the
whole exact forward, and serves to study its convergence.
"""
from __future__ import annotations

import math

import torch

import paper_2609_39034_amd as sw

DEVICE = "cuda"
DECODES = ("decode", "decode_temporal", "decode_gated", "decode_gated_temporal")


def _case(kind, B, H, T, Dk, Dv, J, dtype, *, carry=False, recur=False, name=None):
    c = dict(kind=kind, B=B, H=H, T=T, Dk=Dk, Dv=Dv, J=J, dtype=dtype, carry=carry, recur=recur)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one short sequence of one head in fp32, where the launch and the
        # chain of dependent tokens are all there is
        _case("forward", 1, 1, 64, 16, 16, 2, "f32", name="forward_tiny_f32"),
        # the small training batch (head size 64, four components)
        _case("forward", 4, 8, 2048, 64, 64, 4, "bf16", name="forward_small_bf16"),
        # the language-model batch: the largest whole-sequence call
        _case("forward", 8, 16, 4096, 128, 128, 4, "bf16", name="forward_lm_bf16"),
        # long-context recall: few long sequences of recurring tokens, eight components
        _case("forward", 2, 8, 16384, 128, 128, 8, "bf16", recur=True, name="forward_recall_bf16"),
        # fp32 activations, a later segment of odd length
        _case("forward", 2, 8, 1021, 64, 64, 4, "f32", carry=True, name="forward_segment_f32"),
        # Temporal SwiLA on the small batch, a later segment of odd length
        _case("temporal", 4, 8, 2043, 64, 64, 4, "bf16", carry=True, name="temporal_segment_bf16"),
        # Gated SwiLA, the form of the language models
        _case("gated", 4, 8, 2048, 64, 64, 4, "bf16", name="gated_small_bf16"),
        # Gated Temporal SwiLA on the same batch
        _case("gated_temporal", 4, 8, 2048, 64, 64, 4, "bf16", name="gated_temporal_bf16"),
        # the training step's gradient on the small batch
        _case("backward", 4, 8, 2048, 64, 64, 4, "bf16", name="backward_small_bf16"),
        # gradients in fp32 on a small odd-sized problem
        _case("backward", 2, 4, 509, 32, 64, 4, "f32", carry=True, name="backward_odd_f32"),
        # serving: one token for each of 256 sequences
        _case("decode", 256, 16, 1, 128, 128, 4, "bf16", carry=True, name="decode_batch_bf16"),
        # interactive generation: one token for a handful of sequences
        _case("decode_gated_temporal", 4, 16, 1, 64, 64, 4, "bf16", carry=True,
              name="decode_few_gated_temporal"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


#: state elements times tokens of one head of the largest listed case, over all heads
_MOST = 8 * 16 * 4096 * 4 * 128 * 128


def draw(rng):
    kind = rng.choice(("forward", "forward", "forward", "temporal", "gated", "gated_temporal",
                       "backward", "backward") + DECODES)
    dtype = rng.choice(("bf16", "bf16", "f32"))
    Dk = rng.choice((16, 32, 64, 64, 128, 128))
    Dv = Dk if rng.random() < 0.7 else rng.choice((16, 32, 64, 128))
    J = rng.choice((1, 2, 3, 4, 4, 4, 8))
    H = rng.choice((1, 2, 3, 4, 6, 8, 12, 16))
    carry = rng.random() < 0.5
    if kind in DECODES:
        return _case(kind, _log(rng, 1, 256), H, 1, Dk, Dv, J, dtype, carry=True)
    if kind == "backward":
        T, B, most = _log(rng, 33, 2048), _log(rng, 1, 8), _MOST // 32
    elif dtype == "f32":
        T, B, most = _log(rng, 17, 2048), _log(rng, 1, 8), _MOST // 16
    else:
        T, B, most = _log(rng, 17, 16384), _log(rng, 1, 8), _MOST
    if rng.random() < 0.4 and T >= 64:
        T = T // 64 * 64
    T = min(T, max(17, most // (B * H * J * Dk * Dv)))
    return _case(kind, B, H, T, Dk, Dv, J, dtype, carry=carry,
                 recur=kind == "forward" and rng.random() < 0.25)


def _tdt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def prepare(case, seed):
    """N(0,1) activations and logits with unit keys, as the layer's projections and its key
    normalisation give them; decay logits N(2,1); carried states N(0, 0.1^2) and carried priors that
    are distributions over the components."""
    B, H, T, Dk, Dv, J = (case[n] for n in ("B", "H", "T", "Dk", "Dv", "J"))
    kind, dt = case["kind"], _tdt(case)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    lead = (B, H) if kind in DECODES else (B, T, H)
    ids = torch.randint(0, 1024, (B, T), device=DEVICE, generator=g) if case["recur"] else None

    def normal(*tail):
        if ids is None:
            return torch.randn(lead + tail, device=DEVICE, generator=g)
        return torch.randn((1024, H) + tail, device=DEVICE, generator=g)[ids]

    s = {"case": dict(case)}
    q, k = normal(Dk), normal(Dk)
    k = k / k.norm(dim=-1, keepdim=True).clamp_min(1e-12)
    s["ins"] = [q.to(dt), k.to(dt), normal(Dv).to(dt)] + [normal(J, Dv).to(dt) for _ in range(3)]
    del q, k
    s["state"] = None
    if case["carry"]:
        s["state"] = torch.randn((B, H, J, Dk, Dv), device=DEVICE, generator=g) * 0.1
    if "temporal" in kind:
        s["gates"] = [normal(Dv).to(dt) for _ in range(2)]
        s["prior"] = None
        if case["carry"]:
            s["prior"] = torch.softmax(
                torch.randn((B, H, 2, J, Dv), device=DEVICE, generator=g), dim=3)
    if "gated" in kind:
        s["decay"] = (normal(J, Dk) + 2.0).to(dt)
    if kind == "backward":
        s["grad_o"] = normal(Dv).to(dt)
    return s


def run(state):
    kind, ins, w0 = state["case"]["kind"], state["ins"], state["state"]
    if kind == "forward":
        o, w = sw.forward(*ins, w0)
        return {"o": o, "state": w}
    if kind == "temporal":
        o, w, p = sw.forward_temporal(*ins, *state["gates"], w0, state["prior"])
        return {"o": o, "state": w, "prior": p}
    if kind == "gated":
        o, w = sw.forward_gated(*ins, state["decay"], w0)
        return {"o": o, "state": w}
    if kind == "gated_temporal":
        gk, gq = state["gates"]
        o, w, p = sw.forward_gated(*ins, state["decay"], w0, gate_k_logit=gk, gate_q_logit=gq,
                                   prior_in=state["prior"])
        return {"o": o, "state": w, "prior": p}
    if kind == "backward":
        grads = sw.backward(*ins, w0, state["grad_o"])
        return dict(zip(("dq", "dk", "dv", "dbeta", "dprior_k", "dprior_q", "dstate"), grads))
    if kind == "decode":
        o, w = sw.decode_step(*ins, w0)
        return {"o": o, "state": w}
    if kind == "decode_temporal":
        o, w, p = sw.decode_step_temporal(*ins, *state["gates"], w0, state["prior"])
        return {"o": o, "state": w, "prior": p}
    if kind == "decode_gated":
        o, w = sw.decode_step_gated(*ins, state["decay"], w0)
        return {"o": o, "state": w}
    gk, gq = state["gates"]
    o, w, p = sw.decode_step_gated(*ins, state["decay"], w0, gate_k_logit=gk, gate_q_logit=gq,
                                   prior_in=state["prior"])
    return {"o": o, "state": w, "prior": p}


def work(case):
    B, H, T, Dk, Dv, J = (case[n] for n in ("B", "H", "T", "Dk", "Dv", "J"))
    kind, size = case["kind"], 2 if case["dtype"] == "bf16" else 4
    heads, rows = B * H, B * H * T
    w, prior = 4 * heads * J * Dk * Dv, 4 * heads * 2 * J * Dv
    ins = rows * (2 * Dk + Dv + 3 * J * Dv) * size
    ins += rows * 2 * Dv * size if "temporal" in kind else 0
    ins += rows * J * Dk * size if "gated" in kind else 0
    ins += (w + (prior if "temporal" in kind else 0)) if case["carry"] else 0
    if kind == "backward":
        ins += rows * Dv * size
        outs = 4 * rows * (2 * Dk + Dv + 3 * J * Dv) + w
        return {"bytes": ins + outs, "flops": rows * 2 * 10 * Dk * J * Dv}
    outs = rows * Dv * size + w + (prior if "temporal" in kind else 0)
    per = 2 * 3 * Dk * J * Dv + (Dk * J * Dv if "gated" in kind else 0)
    return {"bytes": ins + outs, "flops": rows * per}


def tolerance(case):
    """bf16 outputs carry the rounding of o to 8 bits (1.7e-3 in the 2-norm against 64 bits).  The
    bf16 backward returns fp32 gradients whose products split fp32 operands into bf16 high parts
    and residuals (5e-6 measured, growing with the sequence); fp32 calls sum over keys and tokens
    in 32 bits (2e-7 to 8e-7 measured, growing with the sequence)."""
    if case["kind"] == "backward":
        return {"rel": 4e-5 if case["dtype"] == "bf16" else 1e-5}
    return {"rel": 8e-3 if case["dtype"] == "bf16" else 1e-5}


def _tokens(x, T):
    """[B,T,H,...] or [B,H,...] inputs as a function of the token."""
    x = x.detach()
    return (lambda t: x.double()) if T is None else (lambda t: x[:, t].double())


def _eq(k):
    return k[:, :, None, :, None]


@torch.no_grad()
def exact(case, seed):
    s = prepare(case, seed)
    B, H, T, Dk, Dv, J = (case[n] for n in ("B", "H", "T", "Dk", "Dv", "J"))
    kind, f64 = case["kind"], dict(device=DEVICE, dtype=torch.float64)
    one = None if kind in DECODES else T
    q, k, v, lb, lk, lq = (_tokens(x, one) for x in s["ins"])
    w = torch.zeros((B, H, J, Dk, Dv), **f64) if s["state"] is None else s["state"].double()
    temporal = "temporal" in kind
    if temporal:
        gk, gq = (_tokens(x, one) for x in s["gates"])
        pr = torch.full((B, H, 2, J, Dv), 1.0 / J, **f64) if s["prior"] is None else s["prior"].double()
        r, rho = pr[:, :, 0], pr[:, :, 1]
    decay = _tokens(s["decay"], one) if "gated" in kind else None
    steps = 1 if one is None else T
    o = torch.empty((steps, B, H, Dv), **f64)
    keep = []
    for t in range(steps):
        kt, qt, vt = k(t), q(t), v(t)[:, :, None]
        if decay is not None:
            w = w * torch.sigmoid(decay(t))[..., None]
        delta = vt - (w * _eq(kt)).sum(3)
        lp = torch.log_softmax(lk(t), 2)
        pq = torch.softmax(lq(t), 2)
        if temporal:
            g = torch.sigmoid(gk(t))[:, :, None]
            lp = torch.log((1 - g) * r + g * lp.exp())
            g = torch.sigmoid(gq(t))[:, :, None]
            rho = (1 - g) * rho + g * pq
            pq = rho
        r = torch.softmax(lp - 0.5 * delta * delta, 2)
        beta = torch.sigmoid(lb(t))
        c = beta * r * delta
        w = w + c[:, :, :, None] * _eq(kt)
        if kind == "backward":
            keep.append((delta, r, c))
            continue
        o[t] = (pq * (w * _eq(qt)).sum(3)).sum(2)
    if kind != "backward":
        out = {"o": o[0] if one is None else o.movedim(0, 1).contiguous(), "state": w}
        if temporal:
            out["prior"] = torch.stack((r, rho), 2)
        return out
    do_of = _tokens(s["grad_o"], T)
    G = torch.zeros_like(w)
    dq, dk = (torch.empty((B, T, H, Dk), **f64) for _ in range(2))
    dv = torch.empty((B, T, H, Dv), **f64)
    dlb, dlk, dlq = (torch.empty((B, T, H, J, Dv), **f64) for _ in range(3))
    for t in range(T - 1, -1, -1):
        delta, r, c = keep.pop()
        kt, qt, do, beta = k(t), q(t), do_of(t)[:, :, None], torch.sigmoid(lb(t))
        pq = torch.softmax(lq(t), 2)
        y = (w * _eq(qt)).sum(3)
        dlq[:, t] = pq * do * (y - (pq * y).sum(2, keepdim=True))
        dy = do * pq
        dq[:, t] = (w * dy[:, :, :, None]).sum((2, 4))
        G = G + dy[:, :, :, None] * _eq(qt)
        dc = (G * _eq(kt)).sum(3)
        w = w - c[:, :, :, None] * _eq(kt)
        dlb[:, t] = dc * c * (1 - beta)
        dr = dc * beta * delta
        da = r * (dr - (r * dr).sum(2, keepdim=True))
        dlk[:, t] = da
        dd = dc * beta * r - delta * da
        dv[:, t] = dd.sum(2)
        dk[:, t] = (G * c[:, :, :, None] - w * dd[:, :, :, None]).sum((2, 4))
        G = G - dd[:, :, :, None] * _eq(kt)
    return {"dq": dq, "dk": dk, "dv": dv, "dbeta": dlb, "dprior_k": dlk, "dprior_q": dlq, "dstate": G}
