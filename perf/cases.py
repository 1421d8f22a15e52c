"""The expert layer's workloads for timing: what a program that uses this library calls, from one decode step of a few
tokens to a whole training step of the largest configuration.

A case names the layer's shape (the fields of workloads.Workload), the pass it makes and the options of the calls:

  mode        "serve": inference forward from tokens to layer output (router, top-k, static dispatch, experts without
              saved activations, combine); "step": forward and backward with all gradients
  gate        "router": the trainable gate is inside the pass (x Wr, and its backward in a step);
              "logits": the caller hands the router's logits over
  capacity    rows allocated for expert-order buffers: "bound" = T * min(k, e_cnt), which always suffices without
              looking at the data; "known" = the routed row count plus 5 %, as a program has it that reads the
              counts once and sizes its buffers by them
  accumulate  whether a step adds its weight gradients to existing ones (micro-batches)
"""
import math

import numpy as np
import torch

from paper_2605_11005_amd import binding as B
from paper_2605_11005_amd import workloads as W
from paper_2605_11005_amd.layer import (MoeLayerBuffers, run_backward, run_backward_router, run_forward,
                                        run_forward_router, torch_dtype)

_LAYER = ("index", "T", "d", "E", "e_lo", "e_cnt", "k", "f", "dtype", "gate_mode", "routing", "zipf_s", "bias_std")


def _case(base, mode, gate, capacity="bound", accumulate=False, **sizes):
    wl = base.scaled(**sizes)
    case = {n: getattr(wl, n) for n in _LAYER}
    case.update(mode=mode, gate=gate, capacity=capacity, accumulate=accumulate)
    return case


def _workload(case):
    return W.Workload(name="case", **{n: case[n] for n in _LAYER})


def listed():
    cases = {
        # one decode step of a small serving batch: every launch is short, latency counts
        "serve-decode-t4": _case(W.QWEN3_T2, "serve", "router", T=4),
        # a decode step of a large serving batch on the largest share: its time is reading 2.8 GB of weights
        "serve-decode-t128": _case(W.DSV3, "serve", "router", T=128),
        # prefill of one prompt of odd length, hidden sizes that are no multiples of the tiles
        "serve-prefill-t2047": _case(W.GPTOSS_T2, "serve", "router", T=2047),
        # the all-fp32 configuration that is checked on the CPU, with its trainable gate
        "step-fp32-tiny": _case(W.TINY, "step", "router"),
        # an fp32 layer of a size that one debugs a model with; odd token count, sizes off the tiles
        "step-fp32-t1500": _case(W.TINY, "step", "logits", T=1500, d=520, f=776, E=16, e_cnt=16, index=21),
        # one short sequence through a small share: few tiles per GEMM, gate trained
        "step-deepseek-moe-t4096": _case(W.DSMOE_T2, "step", "router", T=4096),
        # fine-grained experts, the repository's third configuration
        "step-qwen": _case(W.QWEN, "step", "logits", capacity="known"),
        # a micro-batch that adds to existing gradients, odd token count, ragged hidden sizes
        "step-gpt-oss-t9001-acc": _case(W.GPTOSS_T2, "step", "router", accumulate=True, T=9001),
        # a share of the model table at its full token count with the gate trained
        "step-qwen3": _case(W.QWEN3_T2, "step", "router", capacity="known"),
        # few large experts, all local, gate of eight experts trained: the largest pass
        "step-mixtral": _case(W.MIXTRAL, "step", "router"),
        # the headline configuration
        "step-dsv3": _case(W.DSV3, "step", "logits", capacity="known"),
        # the same with half of the slots on two experts and three empty ones
        "step-dsv3-skew": _case(W.SKEW, "step", "logits", capacity="known"),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("decode", "prefill", "fp32", "step", "step", "step"))
    if kind == "fp32":
        E = rng.choice((8, 12, 16, 32))
        e_cnt = rng.choice((E, E, E // 2))
        return _case(W.TINY, "step", rng.choice(("router", "logits")), rng.choice(("bound", "known")), rng.random() < 0.3,
                     index=rng.randrange(20, 1000), T=_log_int(rng, 64, 3000), d=4 * rng.randrange(16, 257),
                     f=4 * rng.randrange(16, 257), E=E, e_cnt=e_cnt, k=rng.choice((1, 2, 4)),
                     gate_mode=rng.randrange(3))
    base = rng.choice((W.QWEN, W.DSMOE_T2, W.GPTOSS_T2, W.QWEN3_T2, W.DSV3, W.MIXTRAL, None))
    if base is None:         # a share of no particular model
        E = rng.choice((8, 16, 32, 64, 96, 128, 256))
        base = W.QWEN.scaled(d=64 * rng.randrange(8, 65), f=64 * rng.randrange(8, 65), E=E, e_cnt=max(4, E // rng.choice((1, 4, 8))),
                             k=rng.choice((1, 2, 4, 8)), zipf_s=rng.choice((0.0, 0.7, 1.0)), gate_mode=rng.randrange(3))
    sizes = dict(index=rng.randrange(20, 1000))
    if kind == "decode":
        return _case(base, "serve", "router", T=_log_int(rng, 1, 256), **sizes)
    if kind == "prefill":
        return _case(base, "serve", "router", T=_log_int(rng, 512, 8192), **sizes)
    if base is W.DSV3 and rng.random() < 0.3:
        base = W.SKEW
    gate = "logits" if base is W.SKEW else rng.choice(("router", "logits"))
    return _case(base, "step", gate, rng.choice(("bound", "known")), rng.random() < 0.3, T=_log_int(rng, 512, 16384), **sizes)


def _bias(wl):
    """Per-expert popularity: what is added to N(0,1) logits (float64 [E])."""
    if wl.routing == "zipf":
        return -wl.zipf_s * np.log(W.expert_rank(wl).astype(np.float64))
    if wl.routing == "bias_normal":
        return np.random.default_rng(wl.index).standard_normal(wl.E) * wl.bias_std
    return np.zeros(wl.E)


def _skew_logits(wl, randn_like):
    """Logits [T,E] of the skew recipe: see workloads.router_logits."""
    hot, empty, cold = (torch.from_numpy(np.asarray(v)).cuda() for v in W.skew_roles(wl))
    rand = lambda *shape: torch.rand(shape, generator=randn_like, device="cuda")  # noqa: E731
    share = wl.k * wl.e_cnt / wl.E
    score = rand(wl.T, wl.E) + 1.0
    score[:, wl.e_lo:wl.e_lo + wl.e_cnt] -= 1.0
    for group in (hot, cold):
        score[:, group] += 2.0 * (rand(wl.T, len(group)) < 0.5 * share / len(group))
    score[:, empty] = -1.0
    chosen = torch.zeros_like(score).scatter_(1, score.topk(wl.k, dim=1).indices, 1.0)
    return 8.0 * chosen - 4.0 + rand(wl.T, wl.E)


class _State:
    pass


def prepare(case, seed):
    wl = _workload(case)
    dt = torch_dtype(wl)
    g = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=dt)  # noqa: E731
    s = _State()
    s.case, s.wl = case, wl
    s.dev = dev = dict(x=randn(wl.T, wl.d), w1=randn(wl.e_cnt, wl.d, wl.f).mul_(wl.d ** -0.5),
                       w3=randn(wl.e_cnt, wl.d, wl.f).mul_(wl.d ** -0.5), w2=randn(wl.e_cnt, wl.f, wl.d).mul_(wl.f ** -0.5))
    if wl.routing == "skew":
        logits = _skew_logits(wl, g)
    else:
        # hidden states have a component that all tokens share; the router turns it into expert popularity
        wr = randn(wl.d, wl.E).mul_(wl.d ** -0.5)
        dev["x"][:, 0] = 4.0
        wr[0] = torch.from_numpy(_bias(wl) / 4.0).cuda().to(dt)
        logits = dev["x"].float() @ wr.float()
    if case["gate"] == "router":
        dev["wr"] = wr
    else:
        dev["logits"] = logits
    cap = wl.T * min(wl.k, wl.e_cnt)
    if case["capacity"] == "known":
        chosen = logits.topk(wl.k, dim=1).indices
        rows = int(((chosen >= wl.e_lo) & (chosen < wl.e_lo + wl.e_cnt)).sum())
        cap = min(cap, rows + rows // 20 + 8)
    s.buf = MoeLayerBuffers(wl, cap=cap, grads=case["mode"] == "step", router=case["gate"] == "router")
    if case["mode"] == "serve":
        s.buf.h1 = s.buf.h3 = None
        s.status = torch.zeros(1, dtype=torch.int32, device="cuda")
    else:
        dev["dy"] = randn(wl.T, wl.d)
        if case["accumulate"]:
            for t in (s.buf.dw1, s.buf.dw3, s.buf.dw2) + ((s.buf.dwr,) if case["gate"] == "router" else ()):
                t.normal_(generator=g)
    return s


def _serve(wl, dev, buf, status):
    """A serving loop's forward: nothing is kept for a backward pass and no workspace is handed over for the plan."""
    B.moe_router_fwd(dev["x"], dev["wr"], buf.logits, buf.ws_router)
    B.moe_route(buf.logits, wl.k, wl.gate_mode, wl.e_lo, wl.e_cnt, buf.topk_idx, buf.topk_w, buf.counts)
    B.moe_dispatch_static(dev["x"], wl.k, buf.topk_idx, None, wl.e_lo, wl.e_cnt, buf.offsets, buf.perm, buf.inv, buf.xp, status)
    B.moe_expert_fwd(buf.xp, buf.offsets, dev["w1"], dev["w3"], dev["w2"], None, None, buf.o, buf.ws_fwd)
    B.moe_combine(buf.o, buf.inv, buf.topk_w, buf.y)


def run(state):
    case, wl, dev, buf = state.case, state.wl, state.dev, state.buf
    router = case["gate"] == "router"
    if case["mode"] == "serve":
        _serve(wl, dev, buf, state.status)
        return {"y": buf.y, "logits": buf.logits, "topk_idx": buf.topk_idx, "topk_w": buf.topk_w}
    if router:
        run_forward_router(wl, dev, buf)
        run_backward_router(wl, dev, buf, case["accumulate"])
    else:
        run_forward(wl, dev, buf)
        run_backward(wl, dev, buf, case["accumulate"])
    out = {n: getattr(buf, n) for n in ("y", "dx", "dw1", "dw3", "dw2", "topk_idx", "topk_w")}
    if router:
        out.update(logits=buf.logits, dwr=buf.dwr)
    else:       # with given logits the whole plan is determined
        out.update(counts=buf.counts, offsets=buf.offsets, inv=buf.inv)
    return out


def _expected_rows(wl):
    """Expected routed rows of each local expert, from a fixed sample of tokens."""
    if wl.routing == "skew":
        hot, _, cold = W.skew_roles(wl)
        share = wl.T * wl.k * wl.e_cnt / wl.E
        return np.array([0.5 * share / len(hot) if e in hot else 0.5 * share / len(cold) if e in cold else 0.0
                         for e in range(wl.e_lo, wl.e_lo + wl.e_cnt)])
    n = 4096
    logits = np.random.default_rng(1).standard_normal((n, wl.E)) + _bias(wl)
    chosen = np.argpartition(-logits, wl.k - 1, axis=1)[:, :wl.k]
    return np.bincount(chosen.ravel(), minlength=wl.E)[wl.e_lo:wl.e_lo + wl.e_cnt] * (wl.T / n)


def work(case):
    """Inputs read once, outputs written once; weights of an expert without rows are not read in the forward."""
    wl = _workload(case)
    size = 2 if wl.dtype == "bf16" else 4
    rows = _expected_rows(wl)
    active = float(np.sum(1.0 - np.exp(-rows)))
    step, router = case["mode"] == "step", case["gate"] == "router"
    weights, tokens, gate = 3 * wl.d * wl.f * size, wl.T * wl.d * size, wl.d * wl.E * size
    bytes_ = 2 * tokens + active * weights + 8 * wl.T * wl.k                     # x, y, weights, top-k
    flops = 6.0 * rows.sum() * wl.d * wl.f
    if router:
        bytes_ += gate + 4 * wl.T * wl.E
        flops += 2.0 * wl.T * wl.d * wl.E
    else:
        bytes_ += 4 * wl.T * wl.E
    if step:
        grads = wl.e_cnt * weights + (gate if router else 0)
        bytes_ += 2 * tokens + grads * (2 if case["accumulate"] else 1)          # dy, dx, gradients
        flops += 12.0 * rows.sum() * wl.d * wl.f + (4.0 * wl.T * wl.d * wl.E if router else 0.0)
    return {"bytes": bytes_, "flops": flops}


def _gates(wl, logits, topk):
    """Gate weights [T,k] of the selected experts; differentiable in the logits."""
    chosen = logits.gather(1, topk)
    if wl.gate_mode == W.GATE_SOFTMAX_RENORM:
        return chosen.softmax(dim=1)
    if wl.gate_mode == W.GATE_SIGMOID_RENORM:
        s = chosen.sigmoid()
        return s / s.sum(dim=1, keepdim=True)
    return logits.softmax(dim=1).gather(1, topk)


def exact(case, seed):
    """The same outputs in float64 from torch's own products, one expert after the other; nothing for the whole numbers."""
    s = prepare(case, seed)
    wl, dev, step, router = s.wl, s.dev, case["mode"] == "step", case["gate"] == "router"
    x = dev["x"].double()
    logits = x @ dev["wr"].double() if router else dev["logits"].double()
    # the ranking is on fp32 logits
    topk = logits.float().topk(wl.k, dim=1).indices
    logits.requires_grad_(step and router)
    w = _gates(wl, logits, topk)
    g = w.detach()
    y = torch.zeros_like(x)
    out = {"y": y, "topk_idx": None, "topk_w": g}
    if router:
        out["logits"] = logits.detach()
    if step:
        dy = dev["dy"].double()
        dx, dgate = torch.zeros_like(x), torch.zeros_like(g)
        old = lambda t: t.double() if case["accumulate"] else torch.zeros(t.shape, dtype=torch.float64, device="cuda")  # noqa: E731
        dw1, dw3, dw2 = old(s.buf.dw1), old(s.buf.dw3), old(s.buf.dw2)
        out.update(dx=dx, dw1=dw1, dw3=dw3, dw2=dw2)
    for e in range(wl.e_cnt):
        t, j = (topk == wl.e_lo + e).nonzero(as_tuple=True)
        if not len(t):
            continue
        w1, w3, w2 = (dev[n][e].double() for n in ("w1", "w3", "w2"))
        xe, ge = x[t], g[t, j].unsqueeze(1)
        h1, h3 = xe @ w1, xe @ w3
        sig = h1.sigmoid()
        a = h1 * sig * h3
        o = a @ w2
        y.index_add_(0, t, ge * o)
        if step:
            dye = dy[t]
            dgate[t, j] = (dye * o).sum(dim=1)
            do = ge * dye
            da = do @ w2.t()
            dh1, dh3 = da * h3 * sig * (1 + h1 * (1 - sig)), da * h1 * sig
            dw2[e] += a.t() @ do
            dw1[e] += xe.t() @ dh1
            dw3[e] += xe.t() @ dh3
            dx.index_add_(0, t, dh1 @ w1.t() + dh3 @ w3.t())
    if step and router:
        (dlogits,) = torch.autograd.grad(w, logits, dgate)
        dx += dlogits @ dev["wr"].double().t()
        out["dwr"] = old(s.buf.dwr) + x.t() @ dlogits
    elif step:
        out.update(counts=None, offsets=None, inv=None)
    return out


def tolerance(case):
    """bf16: h1, h3, a, o, dH1, dH3, dxp and the outputs are each rounded to 8 bits of mantissa between fp32-accumulated
    products; against the same path in 64 bits every output is off by 2.9e-3 to 3.9e-3 (largest element 0.13).  fp32:
    sums of up to a few thousand terms, off by up to 8e-7 (largest element 1.1e-5).  Ranking is on the fp32 logits: exact
    where they are given; where the router's product makes them, logits closer than its rounding may change places."""
    tol = {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 1e-4}
    if case["gate"] == "router":
        tol["differ"] = 1e-3
    return tol
