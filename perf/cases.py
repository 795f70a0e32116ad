"""The work this library is used for, as cases that can be timed and compared.

A case names one call of the public binding (`paper_2602_07616_amd.binding`) and its sizes.  The
listed ones cover what a serving program and its set-up do with the library:

  decode steps    from one token to the batch of 128 that most experts take part in, on the layer
                  shapes of `paper_2602_07616_amd/workloads.py`, in bf16 and fp32, with re-routing,
                  shared experts, a threshold and the residual connection;
  prefill         hundreds to thousands of tokens through the same layer, also at odd sizes and
                  without re-routing;
  routing alone   for programs that run the experts themselves;
  calibration     the expert-similarity matrix, with two of its metrics.

`draw` gives further sizes of the same ranges, among them the entry point `sere_reroute`, the cosine
metric and the other kernels of centered kernel alignment.
"""
from __future__ import annotations

import math

import torch

from paper_2602_07616_amd import binding as B

WEIGHT_STD = 0.02    # router and expert weights, as in workloads.py
TWIN_NOISE = 0.1     # noise of a planted similar expert, relative to WEIGHT_STD
CLUSTER_STD = 0.5    # spread of hidden states around their cluster's centre

# limits of a drawn case: none costs more than the largest listed one
MAX_BF16_FLOPS = 1.6e11
MAX_BF16_WEIGHTS = 2.9e9
MAX_F32_FLOPS = 2.6e9
MAX_F32_WEIGHTS = 3.0e8


def _case(entry, tokens, hidden, experts, top_k, inter, shared=0, dtype="bf16", S=1, rho=0.0, residual=False,
          clusters=0, twins=0, **more):
    return {"entry": entry, "tokens": tokens, "hidden": hidden, "experts": experts, "top_k": top_k, "inter": inter,
            "shared": shared, "dtype": dtype, "S": S, "rho": rho, "residual": residual, "clusters": clusters,
            "twins": twins, **more}


def listed():
    cases = {
        # the smallest layer, in fp32: five launches on 2 MB of weights; what a test or a debugging run does
        "tiny_f32_t8": _case("decode", 8, 256, 16, 2, 128, dtype="f32", S=1, twins=8),
        # one sequence being decoded, through the entry point that needs no workspace
        "qwen3_t1": _case("static", 1, 2048, 128, 8, 768, S=2, twins=32),
        # a small serving batch whose tokens resemble each other: few experts survive
        "qwen3_t32": _case("decode", 32, 2048, 128, 8, 768, S=2, clusters=8, twins=32),
        # a large serving batch of unrelated tokens: most experts are read
        "qwen3_t128": _case("decode", 128, 2048, 128, 8, 768, S=2, twins=32),
        # shared experts, a threshold and the residual connection of a decoder layer
        "dsv2lite_t64": _case("decode", 64, 2048, 64, 6, 1408, shared=2, S=2, rho=0.3, residual=True, clusters=16),
        # few, very wide experts (d_m = 14336): all of them are read
        "mixtral_t64": _case("decode", 64, 4096, 8, 2, 14336, S=1),
        # a chunk of a prompt at sizes that are no power of two, without re-routing
        "odd2880_t777": _case("baseline", 777, 2880, 32, 4, 1472, shared=1, clusters=4, twins=16),
        # a long prompt: every expert has about 128 tokens
        "qwen3_t2048": _case("decode", 2048, 2048, 128, 8, 768, S=2, twins=32),
        # an fp32 layer of ordinary size, with a shared expert
        "f32_t96": _case("decode", 96, 1024, 32, 4, 704, shared=1, dtype="f32", S=2, rho=0.5, twins=8),
        # routing alone with every optional output, as a program asks for it that runs the experts itself
        "route_t1000": _case("route", 1000, 2048, 128, 8, 768, S=2, rho=0.5, clusters=16, twins=32),
        # set-up: similarity of the experts over calibration text of 128 tokens a batch
        "similarity_frobenius": _case("similarity", 128, 2048, 128, 8, 768, twins=32, clusters=8, batches=4, metric="frobenius"),
        # set-up with centered kernel alignment on short batches
        "similarity_cka": _case("similarity", 32, 2048, 60, 4, 1408, twins=15, clusters=8, batches=2, metric="cka_linear"),
    }
    return [{"name": name, **c} for name, c in cases.items()]


# ------------------------------------------------------------------ draws ---
def _log_int(rng, low, high):
    return max(low, min(high, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def _weights(c):
    return (c["experts"] + c["shared"]) * 3.0 * c["hidden"] * c["inter"] * (4 if c["dtype"] == "f32" else 2)


def _ffn_flops(c):
    return 6.0 * c["hidden"] * c["inter"] * c["tokens"] * (c["top_k"] + c["shared"])


def _fits(c):
    if c["entry"] in ("route", "reroute"):
        return c["tokens"] * c["experts"] * c["hidden"] <= 1.1e9
    if c["entry"] == "similarity":
        rows = c["experts"] * c["tokens"] * c["batches"]
        if _weights(c) > (MAX_F32_WEIGHTS if c["dtype"] == "f32" else 1.3e9):
            return False
        if rows * 6.0 * c["hidden"] * c["inter"] > (MAX_F32_FLOPS if c["dtype"] == "f32" else 6.2e11):
            return False
        if c["metric"] == "cosine":
            return rows * c["experts"] * c["hidden"] <= 1.1e9
        if c["metric"].startswith("cka"):
            return rows * c["tokens"] * c["hidden"] <= 1.0e9 and rows * c["tokens"] * c["experts"] <= 1.0e8
        return True
    f32 = c["dtype"] == "f32"
    return (_weights(c) <= (MAX_F32_WEIGHTS if f32 else MAX_BF16_WEIGHTS)
            and _ffn_flops(c) <= (MAX_F32_FLOPS if f32 else MAX_BF16_FLOPS))


def draw(rng):
    while True:
        entry = rng.choice(["decode"] * 10 + ["baseline"] * 2 + ["static"] * 2 + ["route"] * 2 + ["reroute"] + ["similarity"] * 4)
        f32 = entry != "reroute" and rng.random() < 0.2
        hidden = 64 * _log_int(rng, 4, 24 if f32 else 64)
        experts = _log_int(rng, 2, 64 if f32 else 160)
        inter = 64 * _log_int(rng, 2, 16 if f32 else (224 if experts <= 8 else 44))
        top_k = min(experts, rng.choice([1, 2, 2, 4, 4, 6, 8, 8]))
        c = _case(entry, 1, hidden, experts, top_k, inter, shared=rng.choice([0, 0, 0, 1, 2, 4]),
                  dtype="f32" if f32 else "bf16", S=rng.randint(1, max(1, min(top_k, 3))),
                  rho=rng.choice([0.0, 0.0, 0.3, 0.5]), residual=rng.random() < 0.25, clusters=rng.choice([0, 0, 4, 8, 16]),
                  twins=experts // rng.choice([2, 4, 4, 8]))
        if entry == "static":
            c["tokens"] = _log_int(rng, 1, 64)
            # 32 MiB of scratch: rows of h and of the partial down projections
            if c["tokens"] * (top_k + c["shared"]) * 4 * (inter + hidden * ((inter + 2047) // 2048)) > 24e6:
                continue
        elif entry == "similarity":
            c["shared"] = 0
            c["batches"] = rng.randint(1, 4)
            c["metric"] = rng.choice(["frobenius", "frobenius", "cosine", "cka_linear", "cka_rbf", "cka_poly"])
            # the unbiased estimator behind alignment needs tokens enough not to be all noise
            c["tokens"] = _log_int(rng, 24 if c["metric"].startswith("cka") else 4, 128)
        else:
            c["tokens"] = _log_int(rng, 1, 300 if f32 else 4096)
        if _fits(c):
            return c


# ----------------------------------------------------------------- inputs ---
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
_TAGS = {name: i + 1 for i, name in enumerate(
    ("hidden", "which", "centres", "router", "sim", "ids", "gate_up", "down", "shared_gate_up", "shared_down"))}


def _generator(seed, tag, device="cpu"):
    g = torch.Generator(device=device)
    g.manual_seed((seed * 1000003 + _TAGS[tag] * 7919) % (1 << 62))
    return g


def _hidden(c, seed, count):
    """Hidden states: N(0, 1), or Gaussian clusters whose tokens resemble each other (host)."""
    x = torch.randn(count, c["hidden"], generator=_generator(seed, "hidden"))
    if c["clusters"]:
        centres = torch.randn(c["clusters"], c["hidden"], generator=_generator(seed, "centres"))
        which = torch.randint(c["clusters"], (count,), generator=_generator(seed, "which"))
        x = centres[which] + CLUSTER_STD * x
    return x.to(_DTYPE[c["dtype"]])


def _router(c, seed):
    w = WEIGHT_STD * torch.randn(c["experts"], c["hidden"], generator=_generator(seed, "router"))
    return w.to(_DTYPE[c["dtype"]])


def _sim(c, seed):
    """A symmetric similarity matrix: planted similar pairs at 0.9, all others below 0.4 (host)."""
    m = c["experts"]
    low = torch.triu(0.4 * torch.rand(m, m, generator=_generator(seed, "sim")), 1)
    sim = low + low.T
    sim.fill_diagonal_(1.0)
    for i in range(min(c["twins"], m // 2)):
        sim[i, m - 1 - i] = sim[m - 1 - i, i] = 0.9
    return sim


def _ids(c, seed):
    """Ordered expert indices of every token, distinct within a token (host)."""
    score = torch.rand(c["tokens"], c["experts"], generator=_generator(seed, "ids"))
    return torch.argsort(score, dim=1)[:, :c["top_k"]].to(torch.int32).contiguous()


def _experts(c, seed, tag, count, rows, cols, twins):
    """Expert weights on the GPU; the last `twins` experts are the first ones plus noise."""
    g = _generator(seed, tag, "cuda")
    w = torch.empty(count, rows, cols, dtype=_DTYPE[c["dtype"]], device="cuda").normal_(0.0, WEIGHT_STD, generator=g)
    for i in range(min(twins, count // 2)):
        w[count - 1 - i].mul_(TWIN_NOISE).add_(w[i])
    return w


def _all_experts(c, seed):
    dh, dm, sh = c["hidden"], c["inter"], c["shared"]
    return (_experts(c, seed, "gate_up", c["experts"], 2 * dm, dh, c["twins"]),
            _experts(c, seed, "down", c["experts"], dh, dm, c["twins"]),
            _experts(c, seed, "shared_gate_up", sh, 2 * dm, dh, 0) if sh else None,
            _experts(c, seed, "shared_down", sh, dh, dm, 0) if sh else None)


def _config(c):
    flags = B.SERE_FLAG_RESIDUAL if c["residual"] and c["entry"] in ("decode", "baseline", "static") else 0
    flags |= {"cosine": B.SERE_FLAG_SIM_COSINE, "cka_linear": B.SERE_FLAG_SIM_CKA_LINEAR}.get(c.get("metric"), 0)
    return B.make_config(c["tokens"], c["hidden"], c["experts"], c["top_k"], c["inter"], c["shared"],
                         B.SERE_F32 if c["dtype"] == "f32" else B.SERE_BF16, c["S"], c["rho"], flags)


def _cka_parameters(c):
    """(kernel, param0, param1) of the alignment kernels with parameters: sigma about the distance
    between two outputs of an expert, c about an output's squared norm, cubic polynomial."""
    # an expert's output elements have about this variance for inputs of variance v
    v = 1.0 + CLUSTER_STD ** 2 if c["clusters"] else 1.0
    z = v * c["hidden"] * WEIGHT_STD ** 2                 # variance of a gate and of an up value
    act = 0.25 * z * min(1.0, z) + (0.5 * z if z > 1 else 0.0)
    norm2 = c["hidden"] * c["inter"] * WEIGHT_STD ** 2 * act * z
    if c["metric"] == "cka_rbf":
        return B.SERE_CKA_RBF, math.sqrt(2.0 * norm2), 0.0
    return B.SERE_CKA_POLY, norm2, 3.0


def prepare(case, seed):
    c = dict(case)
    state = {"case": c, "cfg": _config(c)}
    if c["entry"] == "similarity":
        calib = _hidden(c, seed, c["tokens"] * c["batches"]).view(c["batches"], c["tokens"], c["hidden"])
        state["calib"] = calib.cuda()
        state["weights"] = _all_experts(c, seed)
        state["out"] = torch.empty(c["experts"], c["experts"], dtype=torch.float32, device="cuda")
        n = (B.sere_similarity_cka_workspace_bytes if c["metric"] in ("cka_rbf", "cka_poly")
             else B.sere_similarity_workspace_bytes)(state["cfg"], c["tokens"])
        state["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return state
    state["sim"] = _sim(c, seed).cuda()
    if c["entry"] != "static":
        state["workspace"] = B.alloc_workspace(state["cfg"])
    if c["entry"] in ("route", "reroute"):
        state["route"] = B.RouteBuffers.allocate(state["cfg"])
    if c["entry"] == "reroute":
        state["ids"] = _ids(c, seed).cuda()
        return state
    state["hidden"] = _hidden(c, seed, c["tokens"]).cuda()
    state["router"] = _router(c, seed).cuda()
    if c["entry"] != "route":
        state["weights"] = _all_experts(c, seed)
        state["out"] = torch.empty(c["tokens"], c["hidden"], dtype=_DTYPE[c["dtype"]], device="cuda")
    return state


_ROUTE_FIELDS = ("rerouted_ids", "count_before", "count_after", "primary_mask", "num_active", "expert_offsets",
                 "sorted_token", "sorted_slot")


def run(state):
    c, cfg = state["case"], state["cfg"]
    entry = c["entry"]
    if entry == "similarity":
        gu, dn, _, _ = state["weights"]
        if c["metric"] in ("cka_rbf", "cka_poly"):
            kernel, p0, p1 = _cka_parameters(c)
            B.sere_similarity_cka(cfg, state["calib"], c["batches"], c["tokens"], gu, dn, kernel, p0, p1, state["out"],
                                  state["workspace"])
        else:
            B.sere_similarity(cfg, state["calib"], c["batches"], c["tokens"], gu, dn, state["out"], state["workspace"])
        return state["out"]
    if entry == "reroute":
        B.sere_reroute(cfg, state["ids"], state["sim"], state["route"], state["workspace"])
        return {f: getattr(state["route"], f) for f in _ROUTE_FIELDS}
    if entry == "route":
        B.sere_route(cfg, state["hidden"], state["router"], state["sim"], state["route"], state["workspace"])
        return {f: getattr(state["route"], f) for f in ("topk_ids", "topk_weights") + _ROUTE_FIELDS}
    gu, dn, sgu, sdn = state["weights"]
    if entry == "static":
        B.sere_moe_decode_static(cfg, state["hidden"], state["router"], gu, dn, sgu, sdn, state["sim"], state["out"], None)
    elif entry == "baseline":
        B.sere_moe_decode_baseline(cfg, state["hidden"], state["router"], gu, dn, sgu, sdn, state["out"], None,
                                   state["workspace"])
    else:
        B.sere_moe_decode(cfg, state["hidden"], state["router"], gu, dn, sgu, sdn, state["sim"], state["out"], None,
                          state["workspace"])
    return state["out"]


# ------------------------------------------- the same in plain torch, 64 bits ---
def _route_exact(c, hidden, router, sim):
    """(topk_ids, gate weights, rerouted ids) of the batch, in float64."""
    logits = hidden.double() @ router.double().T
    top, ids = torch.sort(logits, dim=1, descending=True, stable=True)
    ids, weights = ids[:, :c["top_k"]], torch.softmax(top[:, :c["top_k"]], dim=1)
    if c["entry"] == "baseline":
        return ids, weights, ids
    return ids, weights, _reroute_exact(c, ids, sim)


def _reroute_exact(c, ids, sim):
    m, S = c["experts"], c["S"]
    primary = torch.zeros(m, dtype=torch.bool, device=ids.device)
    primary[ids[:, :S].reshape(-1)] = True
    masked = torch.where(primary[None, :], sim.double(), torch.tensor(-math.inf, dtype=torch.float64, device=ids.device))
    best = masked.max(dim=1, keepdim=True).values
    first = (masked == best).to(torch.int32).argmax(dim=1)      # the lowest index among equals
    own = torch.arange(m, device=ids.device)
    keep = primary | ((best[:, 0].float() < torch.tensor(c["rho"], dtype=torch.float32)) if c["rho"] > 0 else torch.zeros_like(primary))
    remap = torch.where(keep, own, first)
    new = remap[ids]
    new[:, :S] = ids[:, :S]
    return new


def _expert_exact(x, gate_up, down):
    gu = gate_up.double()
    dm = gu.shape[0] // 2
    g, u = x @ gu[:dm].T, x @ gu[dm:].T
    return (torch.nn.functional.silu(g) * u) @ down.double().T


def _similarity_exact(c, seed):
    m, n, batches = c["experts"], c["tokens"], c["batches"]
    calib = _hidden(c, seed, n * batches).view(batches, n, c["hidden"]).cuda().double()
    gu, dn, _, _ = _all_experts(c, seed)
    total = torch.zeros(m, m, dtype=torch.float64, device="cuda")
    for b in range(batches):
        a = torch.stack([_expert_exact(calib[b], gu[e], dn[e]) for e in range(m)])          # [m, n, d_h]
        if c["metric"] == "frobenius":
            dist = torch.stack([(a - a[p]).square().sum(dim=(1, 2)).sqrt() for p in range(m)])
            total += 1.0 - dist / dist.max()
        elif c["metric"] == "cosine":
            v = (a / a.norm(dim=2, keepdim=True)).reshape(m, -1)
            total += (v @ v.T) / n
        else:
            gram = torch.stack([x @ x.T for x in a])
            if c["metric"] == "cka_rbf":
                _, sigma, _ = _cka_parameters(c)
                d = torch.diagonal(gram, dim1=1, dim2=2)
                gram = torch.exp(-(d[:, :, None] + d[:, None, :] - 2.0 * gram) / (2.0 * sigma * sigma))
            elif c["metric"] == "cka_poly":
                _, offset, degree = _cka_parameters(c)
                gram = (gram + offset) ** int(degree)
            gram = gram * (1.0 - torch.eye(n, dtype=torch.float64, device="cuda"))
            flat, rows = gram.reshape(m, -1), gram.sum(dim=2)
            s = rows.sum(dim=1)
            hsic = flat @ flat.T + torch.outer(s, s) / ((n - 1) * (n - 2)) - 2.0 * (rows @ rows.T) / (n - 2)
            own = torch.diagonal(hsic)
            total += hsic / torch.sqrt(torch.outer(own, own))
    return total / batches


def exact(case, seed):
    c = dict(case)
    if c["entry"] == "reroute":
        return None                       # whole numbers only
    if c["entry"] == "similarity":
        return _similarity_exact(c, seed)
    hidden, router, sim = _hidden(c, seed, c["tokens"]).cuda(), _router(c, seed).cuda(), _sim(c, seed).cuda()
    _, weights, ids = _route_exact(c, hidden, router, sim)
    if c["entry"] == "route":
        return {f: weights if f == "topk_weights" else None for f in ("topk_ids", "topk_weights") + _ROUTE_FIELDS}
    gu, dn, sgu, sdn = _all_experts(c, seed)
    x = hidden.double()
    out = torch.zeros_like(x)
    for e in torch.unique(ids).tolist():
        share = (weights * (ids == e)).sum(dim=1)
        rows = torch.nonzero(share > 0)[:, 0]
        out[rows] += share[rows, None] * _expert_exact(x[rows], gu[e], dn[e])
    for s in range(c["shared"]):
        out += _expert_exact(x, sgu[s], sdn[s])
    return out + x if c["residual"] else out


# ---------------------------------------------------------- work, tolerance ---
def work(case):
    """Each input read once (of the expert weights: those that a batch like this one leaves active), each output written once."""
    c = dict(case)
    eb = 4.0 if c["dtype"] == "f32" else 2.0
    t, dh, dm, m, k = c["tokens"], c["hidden"], c["inter"], c["experts"], c["top_k"]
    expert = 3.0 * dh * dm * eb
    if c["entry"] == "similarity":
        rows = float(t * c["batches"])
        flops = 6.0 * dh * dm * m * rows
        if c["metric"].startswith("cka"):
            flops += m * rows * t * dh + m * m * rows * t      # symmetric matrices: half the products
        else:
            flops += m * m * rows * dh
        return {"bytes": m * expert + rows * dh * eb + 4.0 * m * m, "flops": flops}
    if c["entry"] == "reroute":
        return {"bytes": 4.0 * (t * k * 4 + m * m + 4 * m), "flops": 0.0}
    ids = _route_exact(c, _hidden(c, 1, t), _router(c, 1), _sim(c, 1))
    active = len(torch.unique(ids[2]))
    first = 2.0 * t * m * dh
    total = t * dh * eb + m * dh * eb + (0.0 if c["entry"] == "baseline" else 4.0 * m * (len(torch.unique(ids[0])) - len(torch.unique(ids[0][:, :c["S"]]))))
    if c["entry"] == "route":
        return {"bytes": total + 4.0 * (t * k * 5 + 4 * m), "flops": first}
    return {"bytes": total + (active + c["shared"]) * expert + t * dh * eb, "flops": first + _ffn_flops(c)}


def tolerance(case):
    """About four times what a call shows against `exact` over the listed sizes and thirty drawn ones."""
    if case["entry"] == "reroute":
        return "exact"
    if case["entry"] == "route":
        return {"rel": 2e-7, "max": 1e-6, "differ": 0.0}   # gate weights in fp32, indices the same
    if case["entry"] == "similarity":
        # seen: fp32 layers 2e-8, bf16 layers 3.3e-4 (a bf16 intermediate in the experts)
        return {"rel": 1e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 1.5e-3, "max": 5e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 4e-6}                   # seen: 1.8e-7, 8e-7
    return {"rel": 1e-2, "max": 5e-2}                       # seen: 2.4e-3, 1.3e-2 (bf16 intermediate and output)
