"""The calls whose speed is tracked: what a program that trains or serves one
Pr^2 MoE layer does through the binding, from one decode step of a few
sequences to a training pass over a whole rollout batch.

A case is a dict of plain values: the operation ``op``, the layer (``d`` hidden,
``N`` experts, ``k`` routed per token, ``m`` expert width, ``r`` predictor rank),
``T`` tokens, the activations' type ``act``, the route record's type ``idx``, the
weighting ``renorm`` and the expert load ``skew`` (none, hot8: +1 on the router
bias of eight experts, zipf: a Zipf(1.1) prior).

Layers: the ones of the paper's models that this repository measures or lists
(Qwen3-30B-A3B 2048/128/8/768, Qwen3-235B-A22B 4096/128/8/1536, OLMoE-1B-7B
2048/64/8/1024, Moonlight-16B-A3B 2048/64/6/1408 as d/N/k/m), and the fp32 layer of the
correctness workload.  Drawn cases take hidden sizes in multiples of 256, expert
widths in multiples of 128 and any token count; fp32 layers any size.
"""
from __future__ import annotations

import math

import torch

from paper_2606_00395_amd import binding as B

QWEN30 = dict(d=2048, N=128, k=8, m=768, r=16)
QWEN235 = dict(d=4096, N=128, k=8, m=1536, r=32)
OLMOE = dict(d=2048, N=64, k=8, m=1024, r=16)
MOONLIGHT = dict(d=2048, N=64, k=6, m=1408, r=16)
TINY = dict(d=64, N=8, k=2, m=128, r=4)

DECODE_POSITIONS = 64      # positions of the decode record that a route step writes one of


def _case(name, op, layer, T, act="bf16", idx="int32", renorm=True, skew="hot8"):
    return dict(name=name, op=op, T=T, act=act, idx=idx, renorm=renorm, skew=skew, **layer)


def listed():
    return [
        # one decode step's route recording for 256 sequences, after the rollout's first
        # step (the weight split is kept), into a [sequence, position, k] int16 record
        _case("decode_route_256", "route", QWEN30, 256, idx="int16"),
        # the layer output of a decode step when few sequences are still generating
        _case("decode_layer_8", "rollout", QWEN30, 8, idx="int16"),
        # the same with a full decode batch
        _case("decode_layer_256", "rollout", QWEN30, 256, idx="int16"),
        # prompt processing of a ragged batch under the predictive gates
        _case("prefill_layer_4099", "rollout", OLMOE, 4099),
        # replay of recorded routes in a log-probability pass: the headline layer
        _case("replay_16384", "replay", QWEN30, 16384),
        # the same pass of the largest layer, experts loaded very unevenly
        _case("replay_235b_32768", "replay", QWEN235, 32768, skew="zipf"),
        # a training pass: forward keeping the pre-activations, then its backward
        _case("train_16384", "train", QWEN30, 16384),
        # backward alone (pre-activations recomputed) over an odd micro-batch with the
        # weights as the paper prints them (softmax over all experts)
        _case("backward_literal_3001", "backward", OLMOE, 3001, idx="int16", renorm=False),
        # a training pass with a small ragged micro-batch and 1408-wide experts
        _case("train_moonlight_1021", "train", MOONLIGHT, 1021),
        # fp32 training pass of the correctness workload's layer
        _case("train_fp32_256", "train", TINY, 256, act="f32", skew="none"),
        # predictor training on one response's feature cache (KL loss, dA, dB)
        _case("predictor_loss_2048", "predloss", QWEN30, 2048),
        # routing diagnostics of a training batch against the rollout's logits
        _case("diagnostics_16384", "diag", QWEN30, 16384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["route", "rollout", "rollout", "replay", "replay", "train", "train",
                     "backward", "predloss", "diag", "fp32"])
    idx = rng.choice(["int16", "int32"])
    renorm = rng.random() < 0.75
    if op == "fp32":
        N = rng.randint(2, 32)
        return dict(op=rng.choice(["train", "replay", "rollout"]), T=_log_int(rng, 5, 700),
                    d=rng.randint(17, 260), N=N, k=rng.randint(1, min(N, 4)),
                    m=rng.randint(20, 260), r=rng.randint(1, 8), act="f32", idx=idx,
                    renorm=renorm, skew=rng.choice(["none", "hot8"]))
    layer = dict(rng.choice([QWEN30, OLMOE, MOONLIGHT, QWEN235, None, None]) or
                 dict(d=256 * rng.randint(4, 14), N=4 * rng.randint(4, 32), k=rng.choice([2, 4, 6, 8]),
                      m=128 * rng.randint(4, 14), r=rng.choice([4, 8, 16, 32])))
    lo, hi = {"route": (1, 4096), "rollout": (1, 16384), "replay": (100, 32768),
              "train": (200, 16384), "backward": (200, 16384), "predloss": (200, 4096),
              "diag": (500, 32768)}[op]
    if op in ("train", "backward") and layer["m"] % 256:
        hi = 1200
    # no more work than the largest listed case
    cost = {"rollout": 6, "replay": 6, "train": 18, "backward": 16}.get(op, 0)
    if cost:
        most = 6 * 32768 * 8 * 4096 * 1536
        hi = min(hi, most // (cost * layer["k"] * layer["d"] * layer["m"]))
    return dict(op=op, T=_log_int(rng, lo, max(lo, hi)), act="bf16", idx=idx, renorm=renorm,
                skew=rng.choice(["none", "hot8", "zipf"]), **layer)


# ------------------------------------------------------------------ inputs --

def _draws(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return lambda *shape, std=1.0, dt=torch.float32: torch.randn(
        shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dt)


def _expert(rnd, N, a, b, dt):
    w = torch.empty((N, a, b), device="cuda", dtype=dt)
    for e0 in range(0, N, 16):
        w[e0:e0 + 16] = rnd(min(16, N - e0), a, b, std=0.02, dt=dt)
    return w


def _bias(rnd, N, skew):
    if skew == "none":
        return None
    order = torch.argsort(rnd(N))
    beta = torch.zeros(N, device="cuda")
    if skew == "hot8":
        beta[order[:8]] = 1.0
    else:
        beta[order] = -1.1 * torch.log(torch.arange(1, N + 1, device="cuda", dtype=torch.float32))
    return beta


def _recorded(x, W_r, b_r, k, rnd, idx_dtype):
    """A route that was recorded under earlier parameters: the current top-k, the
    last of them replaced by the next expert on about 5 % of the tokens."""
    z = x.double() @ W_r.double()
    if b_r is not None:
        z += b_r.double()
    ranked = torch.argsort(z, dim=1, descending=True, stable=True)
    ids = ranked[:, :k].clone()
    if k < z.shape[1]:
        swap = rnd(x.shape[0]) > 1.645
        ids[swap, k - 1] = ranked[swap, k]
    return torch.sort(ids, dim=1).values.to(idx_dtype).contiguous()


def _inputs(case, seed):
    """The inputs alone (the same in ``prepare`` and ``exact``)."""
    T, d, N, k, m, r = (case[n] for n in ("T", "d", "N", "k", "m", "r"))
    op = case["op"]
    dt = torch.bfloat16 if case["act"] == "bf16" else torch.float32
    it = torch.int16 if case["idx"] == "int16" else torch.int32
    rnd = _draws(seed)
    s = dict(x=rnd(T, d, dt=dt), W_r=rnd(d, N, std=0.02), A=rnd(d, r, std=0.02),
             Bf=rnd(r, N, std=0.02), b_r=_bias(rnd, N, case["skew"]), dt=dt, it=it)
    if op in ("rollout", "replay", "train", "backward"):
        s["W_gate"] = _expert(rnd, N, m, d, dt)
        s["W_up"] = _expert(rnd, N, m, d, dt)
        s["W_down"] = _expert(rnd, N, d, m, dt)
    if op in ("train", "backward"):
        s["dy"] = rnd(T, d, dt=dt)
    if op in ("replay", "train", "backward", "diag"):
        s["idx"] = _recorded(s["x"], s["W_r"], s["b_r"], k, rnd, it)
    if op in ("predloss", "diag"):
        # the rollout's hidden states and router, and the logits it recorded
        h_old = (s["x"].float() + rnd(T, d, std=0.05)).to(dt)
        W_old = s["W_r"] + rnd(d, N, std=0.002)
        p = h_old.double() @ W_old.double()
        if s["b_r"] is not None:
            p += s["b_r"].double()
        s["h_old"], s["p_old"] = h_old, p.float()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    T, d, N, k, m, r = (case[n] for n in ("T", "d", "N", "k", "m", "r"))
    op, rn = case["op"], bool(case["renorm"])
    x = s["x"]
    s.update(op=op, k=k, renorm=rn)
    code = B.PR2_I16 if s["it"] == torch.int16 else B.PR2_I32
    if op == "route":
        s["record"] = torch.zeros((T, DECODE_POSITIONS, k), dtype=s["it"], device="cuda")
        s["gate"] = torch.empty((T, k), device="cuda")
        s["ws"] = B.route_workspace(x, s["W_r"], s["A"], k, code)
        # the rollout's first step forms the weight split that the others read
        B.route_predict(x, s["W_r"], s["b_r"], s["A"], s["Bf"], k, s["record"][:, 0],
                        gate_out=s["gate"], renorm=rn, ws=s["ws"])
    elif op == "rollout":
        s["ids"] = torch.empty((T, k), dtype=s["it"], device="cuda")
        s["gate"] = torch.empty((T, k), device="cuda")
        s["y"] = torch.empty_like(x)
        s["ws"] = B.rollout_workspace(x, s["W_r"], s["A"], s["W_gate"], k, code, rn)
    elif op == "replay":
        s["gate"] = torch.empty((T, k), device="cuda")
        s["y"] = torch.empty_like(x)
        s["ws"] = B.replay_workspace(x, s["idx"], s["W_r"], s["W_gate"], rn)
    elif op in ("train", "backward"):
        s["dx"] = torch.empty_like(x)
        s["dW_r"] = torch.empty((d, N), device="cuda")
        s["db_r"] = torch.empty((N,), device="cuda")
        for n in ("W_gate", "W_up", "W_down"):
            s["d" + n] = torch.empty(s[n].shape, device="cuda")
        s["ws"] = B.backward_workspace(x, s["idx"], s["W_r"], s["W_gate"], rn)
        if op == "train":
            s["y"] = torch.empty_like(x)
            s["gate"] = torch.empty((T, k), device="cuda")
            s["au"] = torch.empty((T * k, 2 * m), dtype=s["dt"], device="cuda")
            s["ws_fwd"] = B.replay_workspace(x, s["idx"], s["W_r"], s["W_gate"], rn)
    elif op == "predloss":
        s["loss"] = torch.empty((1,), device="cuda")
        s["dA"] = torch.empty((d, r), device="cuda")
        s["dB"] = torch.empty((r, N), device="cuda")
        s["kl"] = torch.empty((T,), device="cuda")
        desc = B.make_desc(T, d, N, 1, 0, r, B.PR2_BF16 if s["dt"] == torch.bfloat16 else B.PR2_F32)
        s["ws"] = torch.empty(max(1, B.workspace_bytes(desc, B.OP_PREDICTOR_LOSS)),
                              dtype=torch.uint8, device="cuda")
    elif op == "diag":
        s["cur"] = torch.empty_like(s["idx"])
        s["overlap"] = torch.empty((T,), dtype=torch.int32, device="cuda")
        s["kl"] = torch.empty((T,), device="cuda")
        s["hist"] = torch.empty((k + 1,), dtype=torch.int64, device="cuda")
        desc = B.make_desc(T, d, N, k, 0, 0, B.PR2_BF16 if s["dt"] == torch.bfloat16 else B.PR2_F32,
                           code)
        s["ws"] = torch.empty(max(1, B.workspace_bytes(desc, B.OP_ROUTE_DIAG)), dtype=torch.uint8,
                              device="cuda")
    else:
        raise ValueError(op)
    return s


def run(s):
    op, rn = s["op"], s["renorm"]
    x, W_r, b_r = s["x"], s["W_r"], s["b_r"]
    if op == "route":
        ids = s["record"][:, 1]
        B.route_predict(x, W_r, b_r, s["A"], s["Bf"], s["k"], ids, gate_out=s["gate"], renorm=rn,
                        ws=s["ws"], reuse_split=True)
        return ids, s["gate"]
    if op == "rollout":
        B.moe_rollout_forward(x, W_r, b_r, s["A"], s["Bf"], s["W_gate"], s["W_up"], s["W_down"],
                              s["k"], s["ids"], s["y"], gate_out=s["gate"], renorm=rn, ws=s["ws"])
        return s["ids"], s["gate"], s["y"]
    if op == "replay":
        B.moe_replay_forward(x, s["idx"], W_r, b_r, s["W_gate"], s["W_up"], s["W_down"], s["y"],
                             gate_out=s["gate"], ws=s["ws"], renorm=rn)
        return s["gate"], s["y"]
    if op in ("train", "backward"):
        grads = (s["dx"], s["dW_r"], s["db_r"], s["dW_gate"], s["dW_up"], s["dW_down"])
        if op == "backward":
            B.moe_replay_backward(x, s["idx"], W_r, b_r, s["W_gate"], s["W_up"], s["W_down"],
                                  s["dy"], *grads, ws=s["ws"], renorm=rn)
            return grads
        B.moe_replay_forward_save(x, s["idx"], W_r, b_r, s["W_gate"], s["W_up"], s["W_down"],
                                  s["y"], s["au"], gate_out=s["gate"], ws=s["ws_fwd"], renorm=rn)
        B.moe_replay_backward_saved(x, s["idx"], W_r, b_r, s["W_gate"], s["W_up"], s["W_down"],
                                    s["au"], s["dy"], *grads, ws=s["ws"], renorm=rn)
        return (s["gate"], s["y"]) + grads
    if op == "predloss":
        B.predictor_loss(x, W_r, b_r, s["h_old"], s["p_old"], s["A"], s["Bf"], s["loss"], s["dA"],
                         s["dB"], kl_out=s["kl"], ws=s["ws"])
        return s["loss"], s["dA"], s["dB"], s["kl"]
    B.route_diagnostics(x, s["idx"], W_r, b_r, z_ref=s["p_old"], cur_idx_out=s["cur"],
                        overlap_out=s["overlap"], kl_out=s["kl"], hist_out=s["hist"], ws=s["ws"])
    return s["cur"], s["overlap"], s["kl"], s["hist"]


# ------------------------------------------------------- work and tolerance --

def work(case):
    T, d, N, k, m, r = (case[n] for n in ("T", "d", "N", "k", "m", "r"))
    ab = 2 if case["act"] == "bf16" else 4
    ib = 2 if case["idx"] == "int16" else 4
    op = case["op"]
    act, route, gates, router = T * d * ab, T * k * ib, T * k * 4, d * N * 4
    pred = (d + N) * r * 4
    logits = 2 * T * d * N
    # experts that some token routes to, were the load even
    used = N * (1 - (1 - k / N) ** T) if k < N else N
    experts = 3 * used * m * d * ab
    if op == "route":
        return dict(bytes=act + router + pred + route + gates, flops=logits + 2 * T * r * (d + N))
    if op == "rollout":
        return dict(bytes=2 * act + router + pred + route + gates + experts,
                    flops=logits + 2 * T * r * (d + N) + 6 * T * k * d * m)
    if op == "replay":
        return dict(bytes=2 * act + router + route + gates + experts,
                    flops=logits + 6 * T * k * d * m)
    if op in ("train", "backward"):
        grads = 3 * N * m * d * 4 + router + N * 4
        n = 18 if op == "train" else 16      # six products of the backward, and a, u (and the output)
        fwd = act + gates if op == "train" else 0
        return dict(bytes=3 * act + fwd + router + route + experts + grads,
                    flops=logits + 4 * T * k * d + n * T * k * d * m)
    if op == "predloss":
        return dict(bytes=2 * act + T * N * 4 + router + 2 * pred + 4 * T,
                    flops=logits + 2 * T * r * (2 * d + 3 * N))
    return dict(bytes=act + router + T * N * 4 + 2 * route + 8 * T, flops=logits)


def tolerance(case):
    # fp32 results (weights, losses, divergences: 2e-7 to 5e-7 seen) come from sums kept to
    # fp32; bf16 layers round H, the weighted expert rows and the result to bf16 on
    # the way (4e-3 per rounding).  ``differ`` is for ids whose logits tie to 1e-6.
    if case["act"] == "f32" or case["op"] in ("route", "predloss", "diag"):
        return {"rel": 3e-6, "max": 1e-3, "differ": 1e-3}
    return {"rel": 1.2e-2, "max": 0.5, "differ": 1e-3}


# ------------------------------------------------------------------- exact --

def _logits(x, W_r, b_r):
    p = x.double() @ W_r.double()
    return p if b_r is None else p + b_r.double()


def _top(z, k):
    """Ids of the k largest fp32 logits, ties to the lower id, ascending."""
    ranked = torch.argsort(z.float(), dim=1, descending=True, stable=True)[:, :k]
    return torch.sort(ranked, dim=1).values


def _gates(z, ids, renorm):
    if renorm:
        return torch.softmax(torch.gather(z, 1, ids), dim=1)
    return torch.gather(torch.softmax(z, dim=1), 1, ids)


def _layer(s, ids, g, dy=None):
    """Layer output; with dy also (dx of the experts, d gate, dW_gate, dW_up, dW_down)."""
    x = s["x"].double()
    T, d = x.shape
    N, m = s["W_gate"].shape[:2]
    y = torch.zeros_like(x)
    if dy is not None:
        dyd = dy.double()
        dx, dg = torch.zeros_like(x), torch.zeros_like(g)
        dWg = torch.zeros((N, m, d), dtype=torch.float64, device=x.device)
        dWu, dWd = torch.zeros_like(dWg), torch.zeros_like(dWg).view(N, d, m)
    for e in range(N):
        t, c = torch.nonzero(ids == e, as_tuple=True)
        if not len(t):
            continue
        X, ge = x[t], g[t, c].unsqueeze(1)
        Wg, Wu, Wd = (s[n][e].double() for n in ("W_gate", "W_up", "W_down"))
        a, u = X @ Wg.T, X @ Wu.T
        sig = torch.sigmoid(a)
        h = a * sig
        H = h * u
        if dy is None:
            y.index_add_(0, t, ge * (H @ Wd.T))
            continue
        O, D = H @ Wd.T, dyd[t]
        y.index_add_(0, t, ge * O)
        dg[t, c] = (D * O).sum(1)
        G = ge * (D @ Wd)
        du, da = G * h, G * u * sig * (1 + a * (1 - sig))
        dx.index_add_(0, t, da @ Wg + du @ Wu)
        dWg[e], dWu[e], dWd[e] = da.T @ X, du.T @ X, D.T @ (ge * H)
    return y if dy is None else (y, dx, dg, dWg, dWu, dWd)


def exact(case, seed):
    s = _inputs(case, seed)
    op, k, rn = case["op"], case["k"], bool(case["renorm"])
    z = _logits(s["x"], s["W_r"], s["b_r"])
    if op in ("route", "rollout"):
        z = z + (s["x"].double() @ s["A"].double()) @ s["Bf"].double()
        ids = _top(z, k)
        g = _gates(z, ids, rn)
        out = (ids.to(s["it"]), g)
        return out if op == "route" else out + (_layer(s, ids, g),)
    if op == "replay":
        ids = s["idx"].long()
        g = _gates(z, ids, rn)
        return g, _layer(s, ids, g)
    if op in ("train", "backward"):
        ids = s["idx"].long()
        g = _gates(z, ids, rn)
        y, dx, dg, dWg, dWu, dWd = _layer(s, ids, g, s["dy"])
        # through the softmax: over the k recorded logits, or over all N
        dp_sel = g * (dg - (g * dg).sum(1, keepdim=True))
        if rn:
            dp = torch.zeros_like(z).scatter_(1, ids, dp_sel)
        else:
            rho = torch.softmax(z, dim=1)
            dp = -rho * (g * dg).sum(1, keepdim=True)
            dp.scatter_add_(1, ids, g * dg)
        dx += dp @ s["W_r"].double().T
        grads = (dx, s["x"].double().T @ dp, dp.sum(0), dWg, dWu, dWd)
        return grads if op == "backward" else (g, y) + grads
    if op == "predloss":
        h, A, Bf = s["h_old"].double(), s["A"].double(), s["Bf"].double()
        u = h @ A
        lr, lh = torch.log_softmax(z, dim=1), torch.log_softmax(s["p_old"].double() + u @ Bf, dim=1)
        kl = (lr.exp() * (lr - lh)).sum(1)
        dz = (lh.exp() - lr.exp()) / z.shape[0]
        return kl.mean().reshape(1), h.T @ (dz @ Bf.T), u.T @ dz, kl
    cur = _top(z, k)
    ids = s["idx"].long()
    overlap = (ids.unsqueeze(2) == cur.unsqueeze(1)).sum((1, 2))
    lr, lh = torch.log_softmax(z, dim=1), torch.log_softmax(s["p_old"].double(), dim=1)
    kl = (lr.exp() * (lr - lh)).sum(1)
    return (cur.to(s["it"]), overlap.to(torch.int32), kl,
            torch.bincount(k - overlap, minlength=k + 1))
