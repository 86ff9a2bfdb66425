"""What the library is timed on: the whole calls a speculative-decoding loop makes for a batch of
positions (the laws, the selection and Algorithm 1, or a diagnostic), through the package's public
entry points, from one-position batches to 65 M-token ones.

Notation: p = target, q = draft, w = p / q, r = law of the selected token.  Rows are synthetic:
softmax of normal logits (a language model's head) or a Zipf target over a permuted vocabulary, the
draft being the target's logits with noise, at its own temperature, whole or cut to its top s tokens.
"""
import math

import torch

import paper_2410_18234_amd as mdss

# Work of one pass besides its bytes: a positive-weight token of one draft law needs about 74 operations
# (nine node terms and eight power sums on the way in, a degree-10 polynomial on the way out).
_LAW_FLOPS = 74

_F64 = torch.float64


def _case(name, call, B, V, K=2, rows="llm", s=0, method="expsum", residual=False, philox=False, tail=0):
    """One case.  call: step | pair | tlp | successive | alphabet | diagnostics.  s: the draft's top-s cut
    (step, successive; 0: whole), |Omega_1| (tlp) or |Omega_0| (alphabet).  tail: the truncated LP's."""
    return {"name": name, "call": call, "B": B, "V": V, "K": K, "rows": rows, "s": s, "method": method,
            "residual": residual, "philox": philox, "tail": tail}


def listed():
    return [
        # A toy vocabulary (unit tests of a sampler, byte-level drafts): nothing but launches.
        _case("tiny_64x16", "step", 64, 16),
        # One decode step of a small serving batch with four drafts, uniforms from the device's generator,
        # and rows that are not 16-byte aligned (odd vocabulary).
        _case("decode_8x50257_k4", "step", 8, 50257, K=4, philox=True),
        # The main workload: 256 positions of a 32000-token vocabulary, two drafts.
        _case("llm_256x32000", "step", 256, 32000),
        # A large vocabulary and batch (the largest rows and bytes).
        _case("zipf_512x128256", "step", 512, 128256, rows="zipf"),
        # Three drafts from a top-1024 draft: the truncated setting of the direct K = 3 rule.
        _case("top1024_256x32000_k3", "step", 256, 32000, K=3, s=1024),
        # The pairwise sums, the default method of step().
        _case("exact_256x32000", "step", 256, 32000, method="exact"),
        # Two drafters of different temperature; the residual and its mass asked for (tree verification
        # goes on from the residual).
        _case("pair_256x32000_residual", "pair", 256, 32000, residual=True),
        # The truncated linear program, Omega_2 sorted, two drafters.
        _case("tlp_sorted_256x32000", "tlp", 256, 32000, s=5, rows="two_temps"),
        # Its sort-free variant, identical drafts, an odd vocabulary, a smaller batch.
        _case("tlp_half_96x50257", "tlp", 96, 50257, s=8, tail=1),
        # Three drafts reduced two at a time, from a top-1024 draft.
        _case("successive_256x32000_k3", "successive", 256, 32000, K=3, s=1024),
        # The truncated alphabet (40 tokens) around the importance-weighted path.
        _case("alphabet_256x32000_m40", "alphabet", 256, 32000, s=40),
        # What an evaluation reports per position: the optimum and the rule's own acceptance.
        _case("diagnostics_256x32000", "diagnostics", 256, 32000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["step", "step", "step", "top", "exact", "pair", "tlp", "tlp", "successive", "alphabet",
                       "diagnostics"])
    V = _log_int(rng, 16, 160000) if call == "step" else _log_int(rng, 4000, 130000)
    if rng.random() < 0.4:
        V = max(16, V // 8 * 8)
    if call == "step":
        B = _log_int(rng, 1, min(1024, max(1, 65000000 // V)))
        c = _case("", "step", B, V, K=rng.choice([2, 2, 3, 4, 8]), rows=rng.choice(["llm", "llm", "zipf"]),
                  residual=rng.random() < 0.25, philox=rng.random() < 0.5)
    elif call == "top":
        c = _case("", "step", _log_int(rng, 1, 512), V, K=rng.choice([3, 3, 4]), s=_log_int(rng, 64, 2000),
                  philox=rng.random() < 0.5)
    elif call == "exact":
        V = min(V, 50000)
        B = _log_int(rng, 1, max(1, min(256, int(256.0 * 32000.0 ** 2 / V ** 2))))
        if rng.random() < 0.3:
            c = _case("", "step", B, V, K=3, s=_log_int(rng, 64, 1000), method="exact")
        else:
            c = _case("", "step", B, V, method="exact", residual=rng.random() < 0.3)
    else:
        B = _log_int(rng, 1, min(384, 12000000 // V))
        if call == "pair":
            c = _case("", "pair", B, V, residual=rng.random() < 0.5, method=rng.choice(["expsum", "expsum", "exact"]))
            if c["method"] == "exact":
                c["V"] = V = min(V, 40000)
                c["B"] = min(B, max(1, int(100.0 * 32000.0 ** 2 / V ** 2)))
        elif call == "tlp":
            c = _case("", "tlp", B, V, s=rng.randint(2, 10), tail=rng.choice([0, 1]),
                      rows=rng.choice(["llm", "zipf", "two_temps"]))
        elif call == "successive":
            c = _case("", "successive", B, V, K=rng.choice([2, 3, 4]), s=rng.choice([0, 256, 1024]))
        elif call == "alphabet":
            c = _case("", "alphabet", B, V, s=_log_int(rng, 10, 400), rows=rng.choice(["llm", "zipf"]))
        else:
            c = _case("", "diagnostics", B, V, K=rng.choice([2, 2, 3]), rows=rng.choice(["llm", "zipf"]))
    del c["name"]
    return c


# ------------------------------------------------------------------------------------ inputs
def _inputs(case, seed):
    B, V, K = case["B"], case["V"], case["K"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal():
        return torch.randn((B, V), generator=g, device="cuda", dtype=_F64)

    if case["rows"] == "zipf":
        mass = torch.arange(1, V + 1, device="cuda", dtype=_F64).pow_(-1.1)
        ell = torch.log(mass / mass.sum())[torch.argsort(torch.rand((B, V), generator=g, device="cuda"), dim=1)]
    else:
        ell = 3.0 * normal()
    two = case["call"] == "pair" or case["rows"] == "two_temps"
    p = torch.softmax(ell, 1)
    if two:
        qs = [torch.softmax((ell + normal()) / t, 1) for t in (1.2, 2.0)]
    else:
        qs = [torch.softmax(ell + normal(), 1)]
    if case["s"] and case["call"] in ("step", "successive"):
        top, at = torch.topk(qs[0], min(case["s"], V), dim=1)
        qs = [torch.zeros_like(qs[0]).scatter_(1, at, top / top.sum(1, keepdim=True))]
    qs = [q.float() for q in qs]
    drafts = []
    for q in qs:
        cdf = torch.cumsum(q.double(), 1)
        n = 1 if two else K
        # strictly below the row's mass: the first token whose running sum exceeds the draw has q > 0
        t = torch.rand((B, n), generator=g, device="cuda", dtype=_F64).clamp_(max=1.0 - 2.0 ** -40)
        drafts.append(torch.searchsorted(cdf, t * cdf[:, -1:], right=True).int())
    bits = torch.randint(0, 1 << 24, (B, 8), generator=g, device="cuda")
    u = bits.float() * 2.0 ** -24
    return {"case": case, "p": p.float(), "q": qs[0], "q2": qs[1] if two else None,
            "drafts": torch.cat(drafts, 1).contiguous(), "u": u[:, :3].contiguous(),
            "u_sel": u[:, 3:3 + max(1, K - 1)].contiguous() if K <= 6 else None, "u2": u[:, 6:8].contiguous()}


def prepare(case, seed):
    return _inputs(case, seed)


# ---------------------------------------------------------------------------------- the calls
def run(state):
    c, p, q, drafts, u = state["case"], state["p"], state["q"], state["drafts"], state["u"]
    call = c["call"]
    if c["philox"]:
        u = None
    if call == "step":
        out = mdss.step(p, q, drafts, u, seed=7, offset=1000, s_max=c["s"], want_residual=c["residual"],
                        method=c["method"])
    elif call == "pair":
        out = mdss.step_pair(p, q, state["q2"], drafts, u, want_residual=c["residual"], method=c["method"])
    elif call == "tlp":
        out = mdss.step_truncated_lp(p, q, state["q2"], drafts, s=c["s"], tail=c["tail"], u=u)
    elif call == "successive":
        out = mdss.step_successive(p, q, drafts, u_sel=state["u_sel"], u=u, method=c["method"])
        del out["r"]  # the last of r_stages
    elif call == "alphabet":
        out = mdss.step_alphabet(p, q, drafts, c["s"], u=u, u2=state["u2"])
    else:
        pstar, kstar = mdss.optimal_acceptance(p, q, c["K"])
        r = mdss.induced_dist_expsum(p, q, c["K"])
        out = {"pstar": pstar, "kstar": kstar, "r": r, "accept": mdss.acceptance(p, r)}
    return {k: v for k, v in out.items() if v is not None}


def work(case):
    B, V, K, s = case["B"], case["V"], case["K"], case["s"]
    n = B * V
    rows = 3 if case["call"] == "pair" or case["rows"] == "two_temps" else 2  # read: p and the draft laws
    written, laws = 1, rows - 1                                              # written: r
    support = min(s, V) if case["call"] in ("step", "successive") and s else V
    if case["residual"]:
        written += 1
    if case["call"] == "tlp":
        flops = 8 * n
    elif case["call"] == "diagnostics":
        flops = (_LAW_FLOPS + 12) * n
    elif case["call"] == "alphabet":
        written += 1
        flops = 2 * n + _LAW_FLOPS * B * s
    elif case["call"] == "successive":
        written = K - 1
        flops = _LAW_FLOPS * B * support * (2 * (K - 2) + 1)
    else:
        flops = _LAW_FLOPS * B * support * laws
    return {"bytes": 4 * n * (rows + written), "flops": flops}


def tolerance(case):
    # The laws are sums of positive terms in fp32: 5e-8 to 9e-8 off in the 2-norm, the residual p - r up to
    # 1.6e-7 (measured against exact()).  Decisions are exact but for a uniform within that of an edge; the
    # smallest best prefix (kstar) also moves where neighbouring prefixes agree to an fp64 sum's rounding.
    return {"rel": 6e-7, "differ": 0.02 if case["call"] == "diagnostics" else 0.002}


# --------------------------------------------------------------------------- 64-bit counterparts
# 1 / D = integral of exp(t - D e^t) dt for every denominator D of the laws; the trapezoidal rule at step 1/4
# is off by 2 |Gamma(1 + 8 pi i)| = 2e-16, and the grid is cut where its tails are below 1e-17.
_H = 0.25


def _grid(w, K):
    pos = w[w > 0]
    lo, hi = float(pos.min()), float(pos.max()) * K
    return [k * _H for k in range(math.floor(math.log(1e-17 / hi) / _H), math.ceil(math.log(45.0 / lo) / _H) + 1)]


def _weights(p, q):
    return torch.where(q > 0, p / torch.where(q > 0, q, torch.ones_like(q)), torch.zeros_like(p))


def _law(p, q, K):
    w, acc = _weights(p, q), torch.zeros_like(p)
    for t in _grid(w, K):
        e = torch.exp(w * -math.exp(t))
        S = (q * e).sum(1, keepdim=True)
        acc += e * (K * _H * math.exp(t) * S ** (K - 1))
    zero = (q > 0) & (p == 0)
    q0 = (q * zero).sum(1, keepdim=True)
    return torch.where(zero, q * q0 ** (K - 1), torch.where(q > 0, p * acc, torch.zeros_like(p)))


def _law_pair(p, q1, q2):
    w1, w2, acc = _weights(p, q1), _weights(p, q2), torch.zeros_like(p)
    for t in _grid(torch.stack((w1.amax(1), w2.amax(1), w1.masked_fill(w1 == 0, math.inf).amin(1),
                                w2.masked_fill(w2 == 0, math.inf).amin(1))), 2):
        e1, e2 = torch.exp(w1 * -math.exp(t)), torch.exp(w2 * -math.exp(t))
        f = _H * math.exp(t)
        acc += e1 * (q1 > 0) * (f * (q2 * e2).sum(1, keepdim=True)) + e2 * (q2 > 0) * (f * (q1 * e1).sum(1, keepdim=True))
    zero = p == 0
    z1, z2 = (q1 * zero).sum(1, keepdim=True), (q2 * zero).sum(1, keepdim=True)
    return torch.where(zero, 0.5 * (q1 * z2 + q2 * z1), p * acc)


def _at(x, i):
    return x.gather(1, i.long())


def _choose(ws, u):
    """Index of the smallest i with u W < w_1 + .. + w_i (W > 0 for tokens drafted from a full-support target)."""
    run = torch.cumsum(ws, 1)
    return (u[:, None].double() * run[:, -1:] >= run).sum(1).clamp(max=ws.shape[1] - 1)


def _algorithm1(p, r, y, u):
    """Algorithm 1 with the proposal r in its fp32 storage: token, accepted, residual, mass."""
    r = r.float().double()
    ok = u[:, 1].double() * _at(r, y[:, None])[:, 0] < _at(p, y[:, None])[:, 0]
    res = (p - r).clamp(min=0.0)
    cdf = torch.cumsum(res, 1)
    z = cdf[:, -1]
    t = torch.searchsorted(cdf, u[:, 2:3].double() * z[:, None], right=True)[:, 0]
    return torch.where(ok, y, t), ok.to(torch.uint8), res, z


def _drawn(p, qs, r, drafts, u, residual):
    ws = torch.cat([_at(p, d) / _at(q, d) for q, d in
                    (zip(qs, (drafts[:, :1], drafts[:, 1:])) if len(qs) == 2 else [(qs[0], drafts)])], 1)
    i = _choose(ws, u[:, 0])
    y = _at(drafts, i[:, None])[:, 0].long()
    out, acc, res, mass = _algorithm1(p, r, y, u)
    got = {"sel_index": i.int(), "sel_token": y.int(), "out_token": out.int(), "accepted": acc}
    if residual:
        got.update(residual=res, mass=mass)
    return got


def exact(case, seed):
    st = _inputs(case, seed)
    c, call, K = case, case["call"], case["K"]
    p, q = st["p"].double(), st["q"].double()
    q2 = st["q2"].double() if st["q2"] is not None else None
    drafts, u = st["drafts"], st["u"]
    zero = torch.zeros(case["B"], dtype=torch.int32, device="cuda")
    free = dict.fromkeys(("sel_index", "sel_token", "out_token", "accepted"))
    if call in ("step", "pair"):
        qs = [q] if call == "step" else [q, q2]
        r = _law(p, q, K) if call == "step" else _law_pair(p, q, q2)
        if c["philox"]:  # the device's own uniforms
            out = dict(free)
            if c["residual"]:
                res = (p - r.float().double()).clamp(min=0.0)
                out.update(residual=res, mass=res.sum(1))
        else:
            out = _drawn(p, qs, r, drafts, u, c["residual"])
        return {"r": r, **out, "status": zero}
    if call == "successive":
        laws, y, i = [_law(p, q, 2)], drafts[:, 0].long(), torch.zeros_like(drafts[:, 0])
        for _ in range(K - 2):
            laws.append(_law_pair(p, laws[-1].float().double(), q))
        for j in range(1, K):
            wy = _at(p, y[:, None])[:, 0] / _at(q if j == 1 else laws[j - 2].float().double(), y[:, None])[:, 0]
            x = drafts[:, j].long()
            wx = _at(p, x[:, None])[:, 0] / _at(q, x[:, None])[:, 0]
            keep = st["u_sel"][:, j - 1].double() * (wy + wx) < wy
            y, i = torch.where(keep, y, x), torch.where(keep, i, torch.full_like(i, j))
        out, acc, _, _ = _algorithm1(p, laws[-1], y, u)
        return {"r_stages": torch.stack(laws), "sel_index": i, "sel_token": y.int(), "out_token": out.int(),
                "accepted": acc, "status": zero}
    if call == "alphabet":
        keep = torch.zeros_like(p).scatter_(1, torch.argsort(-p, dim=1, stable=True)[:, :c["s"]], 1.0)
        mass0 = (p * keep).sum(1)
        pt = (p * keep / mass0[:, None]).float()
        r = _law(pt.double(), q, K)
        return {"p_trunc": pt, "mass0": mass0, "r": r, "sel_index": None, "sel_token": None, "z": None,
                "accepted": None, "out_token": None, "kept": None, "status": zero}
    if call == "diagnostics":
        r = _law(p, q, K)
        order = torch.argsort((p / q).float(), dim=1, stable=True)
        P, Q = torch.cumsum(p.gather(1, order), 1), torch.cumsum(q.gather(1, order), 1)
        total = q.sum(1, keepdim=True) ** K
        f = torch.cat((total, P + total - Q ** K), 1)
        return {"pstar": f.amin(1), "kstar": f.argmin(1).int(), "r": r,
                "accept": torch.minimum(p, r.float().double()).sum(1)}
    # truncated LP: the ranking and the acceptance are unique, the weights (and so r on Omega_1 and what is
    # selected) are not
    b = q if q2 is None else q2
    order = torch.argsort((b * q - p).float(), dim=1, stable=True)
    s = min(c["s"], c["V"])
    ps, qa, qb = (x.gather(1, order) for x in (p, q, b))
    if c["tail"] == 0:
        after = [torch.flip(torch.cumsum(torch.flip(x, (1,)), 1), (1,)) - x for x in (qa, qb)]
        r_tail = (qa * qb + qb * after[0] + qa * after[1])[:, s:]
    else:
        r_tail = 0.5 * (qb * qa[:, s:].sum(1, keepdim=True) + qa * qb[:, s:].sum(1, keepdim=True))[:, s:]
    total = torch.minimum(ps[:, s:], r_tail).sum(1)
    A, Bm = qa[:, s:].sum(1, keepdim=True), qb[:, s:].sum(1, keepdim=True)
    po, ao, bo = ps[:, :s], qa[:, :s], qb[:, :s]
    fixed = ao * bo + bo * A + ao * Bm
    room = (po - fixed).clamp(min=0.0)
    total = total + torch.minimum(po, fixed).sum(1)
    # the pairs' masses flow to their tokens, each up to its room: the least cut over token sets T
    pair = ao[:, :, None] * bo[:, None, :]
    pair = torch.triu(pair + pair.transpose(1, 2), 1)
    cut = None
    for T in range(1 << s):
        inside = torch.tensor([(T >> k) & 1 for k in range(s)], device="cuda", dtype=_F64)
        value = room @ inside + (pair * (1.0 - inside[:, None] * inside[None, :])).sum((1, 2))
        cut = value if cut is None else torch.minimum(cut, value)
    return {"r": None, "omega1": order[:, :s].int(), "w": None, "accept_prob": total + cut, **free, "status": None}
