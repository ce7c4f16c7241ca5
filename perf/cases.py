"""The work this framework is used for, as measurable cases.

Every case goes through the public entry points of ``paper_2609_39137_amd`` (``pipeline.RouterStep`` and, where a
program calls the ABI binding itself, ``binding``).  Kinds:

``route``    inference: hidden states routed with a frozen, trained bias.
``step``     one training iteration of one MoE layer: the router matrix (changed by the optimizer) is packed, the batch
             routed, the bias updated by the ID controller, MaxVio/MinVio written.
``qb``       the same iteration with Quantile Balancing, the strongest baseline controller.
``aux``      the same iteration's forward with the auxiliary loss (softmax router and its statistics).
``select``   biased Top-K, gate weights and counts from scores that another program materialised.
``monitor``  what a training program logs after an iteration: all layers' controller updates with diagnostics, and the
             routing entropies of one layer's batch.

Training cases start from the initial controller state (bias 0), so one pass's gate weights do not depend on how a near
tie falls; ``route`` and ``select`` carry a bias as training leaves it.
"""
from __future__ import annotations

import math

import torch

from paper_2609_39137_amd import binding as B
from paper_2609_39137_amd.pipeline import RouterStep

DEV = "cuda"
KI = KD = 6e-3  # the controller's gains in every configuration of this repository
AUX_ALPHA = 0.05
N_COMPONENTS = 32  # the mixture workloads: 32 component means, sigma 0.5
W_STD = 0.02
BIAS_STD = 0.02  # spread of a trained bias (the closed loops end with biases of this size)


def listed():
    return [
        # A decode batch of a serving program: 32 sequences, one token each, the router matrix packed at load time.
        {"name": "route-decode-t32", "kind": "route", "T": 32, "d": 2048, "E": 768, "K": 10, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # A ragged prefill of a smaller pool of wide hidden states, the router matrix as the checkpoint holds it.
        {"name": "route-prefill-t777-e256", "kind": "route", "T": 777, "d": 4096, "E": 256, "K": 8, "dtype": "bf16",
         "packed": False, "x": "normal"},
        # A training microbatch on the skewed Top-5 mixture (the busiest experts get many times the mean load).
        {"name": "step-t4096-k5-mixture", "kind": "step", "T": 4096, "d": 2048, "E": 768, "K": 5, "dtype": "bf16",
         "packed": True, "x": "mixture"},
        # The headline training step: Top-10 of 768.
        {"name": "step-t16384-k10", "kind": "step", "T": 16384, "d": 2048, "E": 768, "K": 10, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # The largest configuration: a 65536-token batch of 4096-wide hidden states.
        {"name": "step-t65536-d4096", "kind": "step", "T": 65536, "d": 4096, "E": 768, "K": 10, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # The tiny fp32 closed loop (parity and controller studies): Top-4 of 64, row-major router matrix.
        {"name": "step-fp32-t4096-e64", "kind": "step", "T": 4096, "d": 256, "E": 64, "K": 4, "dtype": "f32",
         "packed": False, "x": "normal"},
        # The largest pool with a large K and a ragged batch, row-major router matrix.
        {"name": "step-t5003-e1024-k16", "kind": "step", "T": 5003, "d": 1024, "E": 1024, "K": 16, "dtype": "bf16",
         "packed": False, "x": "normal"},
        # Quantile Balancing at the headline shape.
        {"name": "qb-t16384-k10", "kind": "qb", "T": 16384, "d": 2048, "E": 768, "K": 10, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # Quantile Balancing on a long ragged batch of a smaller pool.
        {"name": "qb-t50001-e256-k8", "kind": "qb", "T": 50001, "d": 1024, "E": 256, "K": 8, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # The auxiliary-loss baseline at the headline shape.
        {"name": "aux-t16384-k10", "kind": "aux", "T": 16384, "d": 2048, "E": 768, "K": 10, "dtype": "bf16",
         "packed": True, "x": "normal"},
        # Selection from scores a program materialised itself, headline shape.
        {"name": "select-t16384-k10", "kind": "select", "T": 16384, "E": 768, "K": 10},
        # Logging after an iteration of a 21-layer model.
        {"name": "monitor-l21-t16384", "kind": "monitor", "L": 21, "T": 16384, "E": 768, "K": 10},
    ]


_MOST = 65536 * 4096 * 768  # multiply-adds of the largest listed case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: tokens, hidden size, pool and K over the ranges the entry points are used in."""
    kind = rng.choice(["route", "route", "step", "step", "step", "qb", "aux", "select", "monitor"])
    if kind in ("select", "monitor"):
        E = rng.choice([rng.randint(33, 1024), 64, 128, 256, 512, 768, 1024])
        K = min(E, rng.choice([1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 32]))
        case = {"kind": kind, "T": _log_int(rng, 16, 65536), "E": E, "K": K}
        if kind == "monitor":
            case["L"] = rng.randint(1, 96)
        return case
    dtype = "f32" if kind in ("route", "step") and rng.random() < 0.2 else "bf16"
    d = 64 * _log_int(rng, 4, 64 if dtype == "bf16" else 16)
    E = rng.choice([32 * rng.randint(2, 32), 64, 128, 256, 384, 512, 768, 1024])
    if kind == "aux":
        E = min(E, 768)
    if dtype == "f32":
        E = min(E, 256)
    K = min(rng.choice([1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24]), E - 1)
    lo, hi = {"route": (1, 16384), "step": (64, 65536), "qb": (256, 65536), "aux": (64, 32768)}[kind]
    T = min(_log_int(rng, lo, hi if dtype == "bf16" else 8192), _MOST // (d * E))
    return {"kind": kind, "T": T, "d": d, "E": E, "K": K, "dtype": dtype, "packed": rng.random() < 0.6,
            "x": rng.choice(["normal", "normal", "mixture"])}


# ---------------------------------------------------------------------------- inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _router_inputs(case, seed):
    """Hidden states, router matrix and bias, in plain torch."""
    g = _gen(seed)
    T, d, E = case["T"], case["d"], case["E"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    W = (torch.randn((E, d), generator=g, device=DEV) * W_STD).to(dt)
    x = torch.empty((T, d), dtype=dt, device=DEV)
    if case["x"] == "mixture":
        mu = torch.randn((N_COMPONENTS, d), generator=g, device=DEV)
        p = torch.rand(N_COMPONENTS, generator=g, device=DEV).log().neg() ** 2  # a few heavy components
        label = torch.multinomial(p, T, replacement=True, generator=g)
    for t0 in range(0, T, 8192):
        t1 = min(T, t0 + 8192)
        e = torch.randn((t1 - t0, d), generator=g, device=DEV)
        x[t0:t1] = mu[label[t0:t1]] + 0.5 * e if case["x"] == "mixture" else e
    bias = torch.randn(E, generator=g, device=DEV) * BIAS_STD if case["kind"] == "route" else \
        torch.zeros(E, device=DEV)
    return x, W, bias


def _score_inputs(case, seed):
    """Sigmoid scores of unit-variance logits and a trained bias."""
    g = _gen(seed)
    s = torch.empty((case["T"], case["E"]), device=DEV)
    for t0 in range(0, case["T"], 8192):
        t1 = min(case["T"], t0 + 8192)
        s[t0:t1] = torch.sigmoid(torch.randn((t1 - t0, case["E"]), generator=g, device=DEV))
    return s, torch.randn(case["E"], generator=g, device=DEV) * BIAS_STD, g


def _monitor_inputs(case, seed):
    s, bias, g = _score_inputs(case, seed)
    L, E, T, K = case["L"], case["E"], case["T"], case["K"]
    w = torch.rand((T, K), generator=g, device=DEV) + 0.5
    w = (w / w.sum(1, keepdim=True)).contiguous()
    load = T * K / E * torch.exp(0.5 * torch.randn((L, E), generator=g, device=DEV))
    counts = load.round().to(torch.int32)
    lb = torch.randn((L, E), generator=g, device=DEV) * BIAS_STD
    le = torch.randn((L, E), generator=g, device=DEV) * 0.3
    return s, bias, w, counts, lb, le


def prepare(case, seed):
    kind = case["kind"]
    if kind == "select":
        s, bias, _ = _score_inputs(case, seed)
        return {"kind": kind, "scores": s, "bias": bias, "K": case["K"],
                "idx": torch.empty((case["T"], case["K"]), dtype=torch.int32, device=DEV),
                "w": torch.empty((case["T"], case["K"]), device=DEV),
                "counts": torch.zeros(case["E"], dtype=torch.int32, device=DEV)}
    if kind == "monitor":
        s, bias, w, counts, lb, le = _monitor_inputs(case, seed)
        state = B.ControllerState(case["E"], DEV, layers=case["L"])
        state.bias.copy_(lb)
        state.e_prev.copy_(le)
        return {"kind": kind, "scores": s, "bias": bias, "w": w, "counts": counts, "state": state,
                "cfg": B.ControllerCfg(case["E"], KI, KD),
                "stats": torch.empty((case["L"], 2), dtype=torch.float64, device=DEV),
                "diag": torch.empty((case["L"], 4), dtype=torch.float64, device=DEV),
                "entropy": torch.empty(2, dtype=torch.float64, device=DEV),
                "workspace": torch.empty(int(B.lib().idb_routing_entropy_workspace_bytes()), dtype=torch.uint8,
                                         device=DEV)}
    x, W, bias = _router_inputs(case, seed)
    rs = RouterStep(case["T"], case["d"], case["E"], case["K"], x.dtype, B.ControllerCfg(case["E"], KI, KD))
    rs.state.bias.copy_(bias)
    if case["packed"]:
        rs.pack(W)  # a serving program packs once; a training program keeps the buffer and packs in every step
    if kind == "qb":
        rs.qb_buffers()
    elif kind == "aux":
        rs.aux_buffers()
    return {"kind": kind, "packed": case["packed"], "rs": rs, "x": x, "W": W}


def run(state):
    kind = state["kind"]
    if kind == "select":
        B.idb_select_from_scores(state["scores"], state["bias"], state["K"], state["idx"], state["w"],
                                 state["counts"])
        return {"idx": state["idx"], "w": state["w"], "counts": state["counts"]}
    if kind == "monitor":
        st = state["state"]
        B.idb_controller_update_layers(state["counts"], state["cfg"], st, state["stats"], state["diag"])
        B.idb_routing_entropy(state["w"], state["entropy"], state["scores"], state["bias"], state["workspace"])
        return {"bias": st.bias, "e_prev": st.e_prev, "step": st.step, "stats": state["stats"],
                "diag": state["diag"], "entropy": state["entropy"]}
    rs, x = state["rs"], state["x"]
    W = None if state["packed"] else state["W"]
    if kind == "route":
        rs.route(x, W)
        return {"idx": rs.idx, "w": rs.w, "counts": rs.counts}
    if state["packed"]:
        rs.pack(state["W"])  # the optimizer changed the router matrix
    if kind == "step":
        rs.step(x, W)
        return {"idx": rs.idx, "w": rs.w, "counts": rs.counts, "bias": rs.state.bias, "e_prev": rs.state.e_prev,
                "step": rs.state.step, "stats": rs.stats}
    if kind == "qb":
        rs.qb_step(x, W)
        return {"idx": rs.idx, "w": rs.w, "counts": rs.counts, "bias": rs.state.bias, "stats": rs.stats}
    rs.aux_step(x, W, alpha=AUX_ALPHA)
    return {"idx": rs.idx, "w": rs.w, "counts": rs.counts, "f": rs.aux_f, "P": rs.aux_P, "loss": rs.aux_loss,
            "stats": rs.stats}


# ---------------------------------------------------------------------------- what a pass needs


def work(case):
    T, E, K = case["T"], case["E"], case["K"]
    if case["kind"] == "select":
        return {"bytes": 4 * T * E + 8 * T * K + 8 * E, "flops": 0}
    if case["kind"] == "monitor":
        return {"bytes": 4 * T * E + 4 * T * K + 4 * E + case["L"] * (20 * E + 64), "flops": 0}
    size = 2 if case["dtype"] == "bf16" else 4
    d = case["d"]
    state = {"route": 8 * E, "step": 20 * E, "qb": 12 * E, "aux": 20 * E}[case["kind"]]
    return {"bytes": size * d * (T + E) + 8 * T * K + state, "flops": 2 * T * d * E}


def tolerance(case):
    """About four times what two accumulation orders of the contraction (16x16x32 and 32x32x16 tiles) differ by.

    Gate weights differ by 1e-7 (aux: 6e-7) where the same experts are chosen.  One near tie in about 1e5 choices falls
    the other way: two loads of the pool then differ by one, which moves e and the bias by 1e-3, and with a trained bias
    the gate weights by 7e-6 (3e-5 with Quantile Balancing's larger biases).  Selection from given scores is defined bit
    for bit, and the monitoring values differ only in the entropies' logarithms (3e-9) and fp32 roundings."""
    return {"route": {"rel": 3e-5, "max": 4e-2, "differ": 1e-2},
            "step": {"rel": 5e-3, "max": 1e-1, "differ": 1e-2},
            "qb": {"rel": 1.2e-4, "max": 4e-2, "differ": 1e-2},
            "aux": {"rel": 1e-3, "max": 2e-2, "differ": 1e-2},
            "select": "exact",
            "monitor": {"rel": 2e-7, "max": 1e-6}}[case["kind"]]


# ---------------------------------------------------------------------------- 64-bit values


def _exact_scores(x, W, t0, t1):
    return torch.sigmoid(x[t0:t1].double() @ W.double().T)


def _exact_routing(case, seed):
    """Gate weights in rank order, and for Quantile Balancing the cutoffs and scores, in 64 bits."""
    x, W, bias = _router_inputs(case, seed)
    T, E, K = case["T"], case["E"], case["K"]
    w = torch.empty((T, K), dtype=torch.float64, device=DEV)
    margins = torch.empty((T, E), dtype=torch.float64, device=DEV) if case["kind"] == "qb" else None
    P = torch.zeros(E, dtype=torch.float64, device=DEV)
    counts = torch.zeros(E, dtype=torch.int64, device=DEV)
    for t0 in range(0, T, 8192):
        t1 = min(T, t0 + 8192)
        if case["kind"] == "aux":
            z = x[t0:t1].double() @ W.double().T
            top = z.topk(K, dim=1)
            w[t0:t1] = torch.softmax(top.values, dim=1)
            P += torch.softmax(z, dim=1).sum(0)
            counts += torch.bincount(top.indices.reshape(-1), minlength=E)
            continue
        s = _exact_scores(x, W, t0, t1)
        v = s + bias.double()
        top = v.topk(K + 1 if case["kind"] == "qb" else K, dim=1)
        sel = s.gather(1, top.indices[:, :K])
        w[t0:t1] = sel / sel.sum(1, keepdim=True)
        if margins is not None:
            margins[t0:t1] = s - top.values[:, K:]
    return w, margins, P, counts


def exact(case, seed):
    """The 64-bit values of what ``run`` returns.  Whole numbers, and what follows from them alone (loads, the bias a
    controller makes of them, MaxVio/MinVio), have none: a near tie that falls the other way is no rounding error."""
    T, E, K = case["T"], case["E"], case["K"]
    kind = case["kind"]
    if kind == "select":
        s, bias, _ = _score_inputs(case, seed)
        w = torch.empty((T, K), dtype=torch.float64, device=DEV)
        for t0 in range(0, T, 8192):
            t1 = min(T, t0 + 8192)
            order = torch.sort(s[t0:t1] + bias, dim=1, descending=True, stable=True).indices[:, :K]
            sel = s[t0:t1].double().gather(1, order)
            w[t0:t1] = sel / sel.sum(1, keepdim=True)
        return {"idx": None, "w": w, "counts": None}
    if kind == "monitor":
        s, bias, w, counts, lb, le = _monitor_inputs(case, seed)
        n = counts.double()
        S = n.sum(1, keepdim=True)
        e = (S - E * n) / S
        de = e - le.double()
        gate = (le.double() * de > 0).double()
        b = lb.double() + KI * e + KD * gate * de
        b = b - b.mean(1, keepdim=True)
        stats = torch.cat([(E * n.amax(1, keepdim=True) - S) / S, (S - E * n.amin(1, keepdim=True)) / S], 1)
        m = (E + 9) // 10
        diag = torch.stack([gate.mean(1), n.sort(1, descending=True).values[:, :m].sum(1) / S[:, 0],
                            (n == 0).double().mean(1), (b - lb.double()).abs().mean(1)], 1)
        top = -(w.double() * w.double().log()).sum(1).mean()
        full = 0.0
        for t0 in range(0, T, 8192):
            c = (s[t0:t0 + 8192] + bias).clamp(min=0).double()
            p = c / c.sum(1, keepdim=True)
            full += float(-torch.special.xlogy(p, p).sum())
        return {"bias": b, "e_prev": e, "step": None, "stats": stats, "diag": diag,
                "entropy": torch.tensor([float(top), full / T], dtype=torch.float64)}
    w, margins, P, counts = _exact_routing(case, seed)
    out = {"idx": None, "w": w, "counts": None}
    if kind == "step":
        out.update(bias=None, e_prev=None, step=None, stats=None)
    elif kind == "qb":
        k = (T * (E - K) + E - 1) // E
        out.update(bias=-margins.T.contiguous().sort(1).values[:, k - 1], stats=None)
    elif kind == "aux":
        P = P / T
        out.update(f=None, P=P, loss=AUX_ALPHA * (counts.double() / T * P).sum().reshape(1), stats=None)
    return out
