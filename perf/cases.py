"""Timing cases of the MoE layer through its public entry points (paper_2512_14080_amd.binding).

A case is one call sequence that a program makes on one layer:
  serve  moe_route + moe_fwd: a decode or prefill call; returns O and the router's scores
  train  moe_route (+ moe_round_tokens) + moe_fwd + moe_bwd: one training step of the layer; returns O and every gradient
  route  moe_route on scores the caller computed + moe_round_tokens: the routing alone; returns the routing's arrays
Weights, routing buffers, outputs and workspaces are allocated in prepare(), as a program keeps them between calls.
"""
import math

import torch

from paper_2512_14080_amd import binding as B

_BF16, _F32, _I32 = torch.bfloat16, torch.float32, torch.int32


def _case(name, kind, T, d, n, E, K, m_tile=0, mode="", zipf=0.0, biases=False, static=False):
    """m_tile 0: token choice without rounding.  zipf: exponent of the router bias (0: no bias).  biases: b1 and b2
    with their gradients.  static: moe_fwd_static instead of a caller's workspace."""
    c = {"kind": kind, "T": T, "d": d, "n": n, "E": E, "K": K, "m_tile": m_tile, "mode": mode, "zipf": zipf,
         "biases": biases, "static": static}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one token through the 7B-shaped layer: a single user's decode step, latency and launches only
        _case("serve-7b-t1", "serve", 1, 1536, 256, 128, 8, static=True),
        # a decode batch of 64 on the 1B-shaped layer: nearly every expert has a few rows
        _case("serve-1b-t64", "serve", 64, 1024, 256, 64, 8, static=True),
        # a large decode batch (or a speculative or chunked one) on a 30B-shaped layer: 1.6 GB of expert weights
        _case("serve-30b-t256", "serve", 256, 4096, 512, 128, 8),
        # one prompt of odd length on the 7B size at the middle granularity: about 110 rows an expert
        _case("prefill-7b-t1777", "serve", 1777, 1536, 512, 64, 4),
        # a prefill batch on the coarse-grained layer (8 experts of n = 14336)
        _case("prefill-coarse-t4096", "serve", 4096, 4096, 14336, 8, 2),
        # a short fine-tuning microbatch on the 1B-shaped layer: 256 rows an expert, token choice
        _case("train-1b-t2048", "train", 2048, 1024, 256, 64, 8),
        # sizes off the tuned grid (d an odd multiple of 128, n of 64, E not a power of two, odd T) with all biases and
        # rounding to 64: what an architecture search or a pruned model has
        _case("train-odd-t5003", "train", 5003, 896, 192, 40, 3, m_tile=64, mode="nearest", zipf=0.3, biases=True),
        # the 1B-shaped layer's full microbatch, token choice
        _case("train-1b-t16384", "train", 16384, 1024, 256, 64, 8),
        # the 7B-shaped layer's full microbatch with token rounding: the headline workload
        _case("train-7b-tr", "train", 32768, 1536, 256, 128, 8, m_tile=128, mode="nearest"),
        # high sparsity with Zipf-distributed expert popularity
        _case("train-sparse-tr", "train", 32768, 2048, 128, 256, 8, m_tile=128, mode="nearest", zipf=1.1),
        # the 30B size's full microbatch with token rounding: the largest step
        _case("train-30b-tr", "train", 32768, 4096, 512, 128, 8, m_tile=128, mode="nearest"),
        # routing with token rounding on scores from the caller's own router, at the 1.4B size's microbatch
        _case("route-1.4b-tr", "route", 40960, 768, 256, 128, 8, m_tile=128, mode="nearest"),
    ]


# (d, n, E, K) of the repository's layer shapes
_SHAPES = [(1024, 256, 64, 8), (1536, 256, 128, 8), (2048, 128, 256, 8), (4096, 14336, 8, 2), (768, 256, 128, 8),
           (768, 512, 64, 4), (768, 1024, 32, 2), (1536, 512, 64, 4), (1536, 1024, 32, 2), (4096, 256, 256, 16),
           (4096, 512, 128, 8), (4096, 1024, 64, 4), (4096, 512, 256, 16), (4096, 1024, 128, 8), (4096, 2048, 64, 4),
           (1536, 256, 512, 8), (1536, 1024, 16, 2), (4096, 512, 64, 8)]
_COST_OPS, _COST_BYTES = 1.1e13, 2.5e10  # about the largest listed case's


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choices(["serve", "train", "route"], [5, 6, 1])[0]
        if rng.random() < 0.6:
            d, n, E, K = rng.choice(_SHAPES)
        else:
            d = 128 * rng.randint(3, 32)
            n = 64 * _log_int(rng, 1, 24)
            E = 8 * _log_int(rng, 1, 48)
            K = min(rng.choice([1, 2, 3, 4, 6, 8, 8, 10, 16]), E // 2)
        T = _log_int(rng, 1, 8192) if kind == "serve" else _log_int(rng, 512, 40960)
        m_tile, mode = 0, ""
        if kind == "route" or (kind == "train" and rng.random() < 0.6):
            m_tile = rng.choice([64, 128, 128, 128, 256])
            mode = rng.choice(["nearest", "nearest", "nearest", "up", "down", "balance"])
        c = _case("", kind, T, d, n, E, K, m_tile, mode, zipf=rng.choice([0.0, 0.0, 0.5, 1.1]),
                  biases=kind != "route" and rng.random() < 0.25, static=False)
        if kind == "serve" and not c["biases"]:
            c["static"] = T * K * (n + d) * 2 < (60 << 20) and rng.random() < 0.5
        w = work(c)
        if w["flops"] <= _COST_OPS and w["bytes"] <= _COST_BYTES and 6 * d * n * E <= 8e9:
            return c


def _inputs(case, seed):
    """The tensors of a case: activations of a normalised residual stream (unit variance), weights of standard
    deviation 0.02, a router whose logits have unit variance."""
    T, d, n, E = case["T"], case["d"], case["n"], case["E"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std, dtype=_BF16):
        return torch.randn(shape, generator=g, device="cuda", dtype=dtype).mul_(std)

    s = {"bias": None, "b1": None, "b2": None}
    if case["zipf"]:
        rank = torch.randperm(E, generator=g, device="cuda") + 1
        s["bias"] = -case["zipf"] * rank.to(_F32).log()
    if case["kind"] == "route":
        logits = normal((T, E), 1.0, _F32)
        s["scores"] = torch.softmax(logits if s["bias"] is None else logits + s["bias"], dim=1)
        return s
    s["X"] = normal((T, d), 1.0)
    s["Wr"] = normal((d, E), d ** -0.5)
    s["W1"] = normal((E, d, 2 * n), 0.02)
    s["W2"] = normal((E, n, d), 0.02)
    if case["biases"]:
        s["b1"] = normal((E, 2 * n), 0.1, _F32)
        s["b2"] = normal((E, d), 0.1, _F32)
    if case["kind"] == "train":
        s["dO"] = normal((T, d), 1.0)
    return s


def prepare(case, seed):
    T, d, n, E, K = (case[k] for k in ("T", "d", "n", "E", "K"))
    kind, m_tile = case["kind"], case["m_tile"]
    s = _inputs(case, seed)
    D = s["D"] = B.dims(T, d, n, E, K)
    s.update(kind=kind, m_tile=m_tile, mode=case["mode"], static=case["static"])
    s["tc"] = B.Routing(D, T * K, B.MOE_ROUTING_SCORES_T if m_tile else 0)
    s["flags"] = (B.MOE_ROUTE_WRITE_SCORES_T | B.MOE_ROUTE_COUNTS_ONLY) if m_tile else 0
    s["r"] = s["tc"]
    if m_tile:
        s["r"] = B.Routing(D, B.moe_round_capacity(D, m_tile))
    cap = s["r"].capacity
    if kind == "route":
        s["tc"].buf.zero_()
        s["r"].buf.zero_()  # the rows past the routed ones are never written
        s["tc"].arrays()["scores"].copy_(s.pop("scores"))
        s["flags"] |= B.MOE_ROUTE_SCORES_IN
        a, t = s["r"].arrays(), s["tc"].arrays()
        s["out"] = {k: a[k] for k in ("mask", "counts", "offsets", "row_token", "row_expert", "row_w", "tok_offsets",
                                      "tok_rows", "tok_count", "round_dir")}
        s["out"].update(topk_idx=t["topk_idx"], topk_w=t["topk_w"], scores_t=t["scores_t"])
        return s

    def empty(*shape, dtype=_BF16):
        return torch.empty(shape, dtype=dtype, device="cuda")

    train = kind == "train"
    s["H"], s["O"] = empty(cap, 2 * n), empty(T, d)
    s["out"] = {"O": s["O"]}
    if not train:
        s["out"]["scores"] = s["tc"].arrays()["scores"]
    db1 = db2 = None
    if train:
        for k, t in (("dX", empty(T, d)), ("dW1", empty(E, d, 2 * n)), ("dW2", empty(E, n, d)),
                     ("dWr", empty(d, E, dtype=_F32)), ("dbias", empty(E, dtype=_F32))):
            s[k] = s["out"][k] = t
        if case["biases"]:
            db1 = s["out"]["db1"] = empty(E, 2 * n, dtype=_F32)
            db2 = s["out"]["db2"] = empty(E, d, dtype=_F32)
        s["ws_b"] = empty(B.moe_workspace_bytes(D, cap, B.MOE_WS_BWD), dtype=torch.uint8)
    if not case["static"]:
        s["ws_f"] = empty(B.moe_workspace_bytes(D, cap, B.MOE_WS_FWD), dtype=torch.uint8)
    s["eb"] = B.expert_bias(s["b1"], s["b2"], db1, db2)
    return s


def run(s):
    D, kind = s["D"], s["kind"]
    B.moe_route(D, s.get("X"), s.get("Wr"), s["bias"] if kind != "route" else None, s["flags"], s["tc"])
    if s["m_tile"]:
        B.moe_round_tokens(D, s["m_tile"], s["mode"], None, s["tc"], s["r"])
    if kind == "route":
        return s["out"]
    if s["static"]:
        B.moe_fwd_static(D, s["X"], s["W1"], s["W2"], s["r"], s["H"], s["O"], eb=s["eb"])
    else:
        B.moe_fwd(D, s["X"], s["W1"], s["W2"], s["r"], s["H"], s["O"], s["ws_f"], eb=s["eb"])
    if kind == "train":
        B.moe_bwd(D, s["dO"], s["X"], s["H"], s["W1"], s["W2"], s["Wr"], s["r"], s["dX"], s["dW1"], s["dW2"],
                  s["dWr"], s["dbias"], None, s["ws_b"], eb=s["eb"])
    return s["out"]


def work(case):
    T, d, n, E, K = (case[k] for k in ("T", "d", "n", "E", "K"))
    P = T * K  # routed rows (rounding keeps their number to within a few per cent)
    if case["kind"] == "route":
        # scores in; transposed scores, selection, bitmap, row lists and token lists out
        return {"bytes": 8 * T * E + 8 * P + T * E / 8 + 12 * P + 4 * P + 8 * T, "flops": 5 * T * E}
    hit = E * (1 - (1 - K / E) ** T)  # experts that at least one token picks
    if case["zipf"]:  # under the skewed router the unpopular ones are picked less often
        p = [r ** -case["zipf"] for r in range(1, E + 1)]
        hit = sum(1 - max(0.0, 1 - K * x / sum(p)) ** T for x in p)
    wbytes = 2 * hit * 3 * d * n  # W1 and W2 of those experts
    byts = 2 * T * d + 2 * d * E + wbytes + 4 * T * E + 4 * P * n + 2 * T * d  # X, W_r, weights; scores, H, O
    flops = 2 * T * d * E + 6 * P * d * n
    if case["kind"] == "train":
        # dO; dX, dW1 and dW2 of every expert, dW_r
        byts += 2 * T * d + 2 * T * d + 6 * E * d * n + 4 * d * E
        flops += 4 * T * d * E + 12 * P * d * n
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "route":
        # the routing is a function of the given scores, ties included; the weights are one fp32 sum and quotient
        return {"rel": 1e-6, "differ": 0.0}
    # bf16 activations between the GEMMs (H, A, Y, dH, A', dX~): every output is 2.5e-3 to 3.9e-3 off the same in 64
    # bits.  A token whose K-th and next scores agree to fp32 rounding may take either expert, which moves its own row
    # of O and dX by up to about its rms.
    return {"rel": 1e-2, "max": 0.95}


# ------------------------------------------------------------------ the same in 64 bits, plain torch
def _select(S, case):
    """Membership [T, E] of token choice, then of token rounding, from scores S."""
    T, E, K, M = case["T"], case["E"], case["K"], case["m_tile"]
    idx = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :K]
    tc = torch.zeros((T, E), dtype=torch.bool, device=S.device)
    tc.scatter_(1, idx, True)
    if not M:
        return idx, tc, None
    f = tc.sum(0).tolist()
    keep, direction, z = [], [], 0
    for c in f:
        lo, hi = c // M * M, -(-c // M) * M
        if case["mode"] == "up":
            pad = True
        elif case["mode"] == "down":
            pad = False
        elif case["mode"] == "balance":
            pad = abs(z + hi - c) < abs(z + lo - c)
        else:
            pad = hi - c < c - lo
        pad = pad and hi <= T
        keep.append(hi if pad else lo)
        z += keep[-1] - c
        direction.append((keep[-1] > c) - (keep[-1] < c))
    key = torch.where(tc, S + 2, S)  # scores are in [0, 1]: chosen tokens first
    order = torch.sort(key, dim=0, descending=True, stable=True).indices
    place = torch.empty_like(order)
    place.scatter_(0, order, torch.arange(T, device=S.device)[:, None].expand(T, E))
    return idx, place < torch.tensor(keep, device=S.device)[None, :], direction


def exact(case, seed):
    T, d, n, E, K = (case[k] for k in ("T", "d", "n", "E", "K"))
    s = _inputs(case, seed)
    f64 = torch.float64
    if case["kind"] == "route":
        S = s["scores"].double()
        idx, member, _ = _select(S, case)
        w = torch.gather(S, 1, idx)
        rw = torch.zeros(min(T * E, T * K + E * (case["m_tile"] - 1)), dtype=f64, device="cuda")
        rows = (S * member / (S * member).sum(1, keepdim=True).clamp_min(1e-300)).t()[member.t()]
        rw[:rows.numel()] = rows
        out = dict.fromkeys(("mask", "counts", "offsets", "row_token", "row_expert", "tok_offsets", "tok_rows",
                             "tok_count", "round_dir", "topk_idx"))
        return {**out, "row_w": rw, "topk_w": w / w.sum(1, keepdim=True), "scores_t": S.t().contiguous()}
    X, Wr = s["X"].double(), s["Wr"].double()
    logits = X @ Wr
    if s["bias"] is not None:
        logits += s["bias"].double()
    S = torch.softmax(logits, 1)
    _, member, _ = _select(S, case)
    sw = S * member
    sw = sw / sw.sum(1, keepdim=True).clamp_min(1e-300)
    O = torch.zeros((T, d), dtype=f64, device="cuda")
    train = case["kind"] == "train"
    out = {"O": O} if train else {"O": O, "scores": S}
    if train:
        dO = s["dO"].double()
        dX, dS = torch.zeros_like(O), torch.zeros((T, E), dtype=f64, device="cuda")
        out.update(dX=dX, dW1=torch.zeros((E, d, 2 * n), dtype=f64, device="cuda"),
                   dW2=torch.zeros((E, n, d), dtype=f64, device="cuda"))
        if case["biases"]:
            out.update(db1=torch.zeros((E, 2 * n), dtype=f64, device="cuda"),
                       db2=torch.zeros((E, d), dtype=f64, device="cuda"))
    for e in range(E):
        t = member[:, e].nonzero()[:, 0]
        if not t.numel():
            continue
        w, x, W1, W2 = sw[t, e][:, None], X[t], s["W1"][e].double(), s["W2"][e].double()
        h = x @ W1
        if case["biases"]:
            h += s["b1"][e].double()
        gate, up = h[:, :n], h[:, n:]
        sig = torch.sigmoid(gate)
        a = gate * sig * up
        y = a @ W2
        if case["biases"]:
            y += s["b2"][e].double()
        O.index_add_(0, t, w * y)
        if not train:
            continue
        do = dO[t]
        da = do @ W2.t()
        dS[t, e] = (do * y).sum(1)
        da *= w
        dh = torch.cat([da * up * sig * (1 + gate * (1 - sig)), da * gate * sig], 1)
        out["dW2"][e] = (w * a).t() @ do
        out["dW1"][e] = x.t() @ dh
        dX.index_add_(0, t, dh @ W1.t())
        if case["biases"]:
            out["db1"][e], out["db2"][e] = dh.sum(0), (w * do).sum(0)
    if train:
        dL = sw * (dS - (sw * dS).sum(1, keepdim=True))
        dX += dL @ Wr.t()
        out.update(dWr=X.t() @ dL, dbias=dL.sum(0))
    return out
