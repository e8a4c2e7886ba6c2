"""The work whose speed is measured: calls of this library as a user's
program makes them, from the smallest batch to the largest, with the inputs
they meet (group sizes, reward types, probability floors and score widths of
the workloads that the tests and the benchmark use).

A case is a dict of plain values.  Its "kind" names the calls:

  step        one training step's estimator: the design draw with the
              coefficient fold, then the per-prompt gradient
  logged      the same from masks and a rho block that were logged earlier,
              with the weight diagnostics (ESS, largest weight)
  mean        the batch-mean gradient of given coefficients
  replicates  design draws of many replicates (masks, counts, rho block)
  audit       the Monte-Carlo audit of a frozen population
  direction   the audit's update-direction column
  exact       the closed-form audit
  alloc       the probability design that precedes a step
  fixed       the fixed-size design: fit of the odds, then draws

Groups have `gmin` .. `gmax` candidates (gmin = gmax: all alike).
"""
import math

import numpy as np
import torch

import paper_2608_11368_amd as pair

DEV = "cuda:0"
PI_MIN = 0.08
RULES = {"ht": pair.RULE_HT, "unweighted": pair.RULE_UNWEIGHTED, "ratio_ke": pair.RULE_RATIO_KE,
         "clipped": pair.RULE_CLIPPED, "selfnorm": pair.RULE_SELFNORM,
         "marginal": pair.RULE_MARGINAL}
WMAX = 10.0


def listed():
    return [
        # The smallest step: four prompts of eight candidates on one small
        # parameter block, fp32 scores.  Launches and host calls count.
        dict(name="step_tiny", kind="step", B=4, gmin=8, gmax=8, D=4096, pad=0, dtype="f32"),
        # The ordinary training step: 128 prompts of 16, 2^20 parameters, bf16.
        dict(name="step_b128", kind="step", B=128, gmin=16, gmax=16, D=1 << 20, pad=0,
             dtype="bf16"),
        # A large step on groups of uneven size, from logged masks and rho,
        # with the weight diagnostics that a run logs.
        dict(name="logged_ragged", kind="logged", B=512, gmin=2, gmax=64, D=1 << 18, pad=0,
             dtype="bf16", rule="ht"),
        # The batch-mean update of fp32 scores whose width is odd, in padded rows.
        dict(name="mean_odd_f32", kind="mean", B=96, gmin=2, gmax=32, D=400003, pad=1,
             dtype="f32"),
        # The draws of an audit matrix: many replicates of a ragged batch.
        dict(name="replicates_ragged", kind="replicates", B=512, gmin=2, gmax=64, R=1000),
        # The frozen-population audit at its full size.
        dict(name="audit_full", kind="audit", B=256, gmin=16, gmax=16, D=65536, pad=0, R=4096,
             rule="ht"),
        # An estimator variant on uneven groups, odd width and replicate count.
        dict(name="audit_ragged", kind="audit", B=64, gmin=2, gmax=64, D=20011, pad=5, R=1000,
             rule="clipped"),
        # The audit as a quick check during development: a handful of prompts.
        dict(name="audit_small", kind="audit", B=4, gmin=8, gmax=8, D=4096, pad=0, R=256,
             rule="ht"),
        # The cosine column of the audit matrix at the audit's full size.
        dict(name="direction_full", kind="direction", B=256, gmin=16, gmax=16, D=65536, pad=0,
             R=4096, rule="ht"),
        # The closed-form audit of a ragged batch.
        dict(name="exact_ragged", kind="exact", B=128, gmin=2, gmax=64, D=65536, pad=0,
             rule="ht"),
        # The probability design that a step starts with, for a large batch.
        dict(name="alloc_ragged", kind="alloc", B=512, gmin=2, gmax=64),
        # The fixed-size design of a large batch: fit, then replicate draws.
        dict(name="fixed_ragged", kind="fixed", B=512, gmin=2, gmax=64, R=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "logged", "mean", "replicates", "audit", "audit", "direction",
                       "exact", "alloc", "fixed"])
    B = _log_int(rng, 4, 512)
    gmax = rng.choice([8, 16, 64, rng.randint(2, 64)])
    gmin = gmax if rng.random() < 0.5 else rng.randint(2, gmax)
    c = dict(kind=kind, B=B, gmin=gmin, gmax=gmax)
    rows = B * (gmin + gmax) // 2
    if kind in ("alloc", "fixed", "replicates"):
        if kind != "alloc":
            most = 16_000_000 if kind == "replicates" else 4_000_000
            c["R"] = _log_int(rng, 16, max(16, min(4096, most // rows)))
        return c
    mc = kind in ("audit", "direction")
    dtype = rng.choice(["bf16", "bf16", "f32"]) if kind in ("step", "logged", "mean") else "bf16"
    wide = (1 << 18) if mc or kind == "exact" else (1 << 20)
    most = min(wide, (1 << 31) // rows)
    if mc:
        c["R"] = _log_int(rng, 64, 4096)
        most = min(most, int(1e12 / (rows * c["R"])))
    D = _log_int(rng, 512, max(512, most))
    D = D if rng.random() < 0.5 else max(512, D - D % 512)
    unit = 8 if dtype == "bf16" else 4
    c.update(D=D, pad=-D % unit, dtype=dtype)
    if kind in ("audit", "direction", "logged"):
        c["rule"] = rng.choice(list(RULES))
    elif kind == "exact":
        c["rule"] = rng.choice(["ht", "unweighted", "clipped", "marginal"])
    return c


# ------------------------------------------------------------------ inputs --
def _sizes(case):
    """Group sizes: a fixed cycle over gmin .. gmax, so that every seed of a
    case has the same work; the seed decides their order."""
    lo, hi, B = case["gmin"], case["gmax"], case["B"]
    return lo + (np.arange(B, dtype=np.int64) * (hi - lo + 1)) // B


def _host(case, seed):
    """Sizes, offsets, rewards and continuation probabilities on the host."""
    rng = np.random.default_rng(seed)
    sizes = rng.permutation(_sizes(case))
    off = np.zeros(case["B"] + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    nv = int(off[-1])
    owner = np.repeat(np.arange(case["B"]), sizes)
    if case["gmin"] == case["gmax"]:
        # verifiable rewards, one success rate per prompt (some prompts saturate)
        q = rng.beta(0.5, 0.5, case["B"])
        rewards = (rng.random(nv) < q[owner]).astype(np.float32)
    else:
        rewards = rng.random(nv).astype(np.float32)   # partial credit
    p = np.minimum(rng.uniform(0.1, 1.0, nv).astype(np.float32), np.float32(1.0))
    return dict(rng=rng, sizes=sizes, off=off, nv=nv, owner=owner, rewards=rewards, p=p)


def _up(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _scores(case, nv, seed):
    """Score rows N(0, 1/D) (unit variance for fp32), drawn on the GPU; the
    padding of a row holds NaN, which no call may read."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 7919)
    D, f32 = case["D"], case.get("dtype") == "f32"
    full = torch.empty((nv, D + case["pad"]), dtype=torch.float32 if f32 else torch.bfloat16,
                       device=DEV)
    step = max(1, (1 << 28) // D)
    for r in range(0, nv, step):
        blk = full[r:r + step, :D]
        blk.normal_(generator=gen)
        if not f32:
            blk.mul_(1.0 / math.sqrt(D))
    if case["pad"]:
        full[:, D:] = float("nan")
    return full[:, :D]


def _logged(case, h):
    """A mask and its logged rho block, from torch on the host's numbers."""
    B, g = case["B"], case["gmax"]
    pp = np.zeros((B, g), dtype=np.float32)
    pos = np.arange(h["nv"]) - h["off"][:-1][h["owner"]]
    pp[h["owner"], pos] = h["p"]
    pi = pp[:, :, None] * pp[:, None, :]
    d = np.arange(g)
    pi[:, d, d] = pp
    mask = (h["rng"].random(h["nv"]) < h["p"]).astype(np.uint8)
    return mask, pi


def prepare(case, seed):
    h = _host(case, seed)
    kind, B = case["kind"], case["B"]
    s = dict(case=case, kind=kind, B=B, gmax=case["gmax"], nv=h["nv"], off=_up(h["off"]),
             seed=int(seed))
    if kind == "alloc":
        p_hat = h["rng"].uniform(0.02, 0.98, h["nv"]).astype(np.float32)
        c_hat = h["rng"].lognormal(math.log(4000.0) - 0.5, 1.0, h["nv"]).astype(np.float32)
        budget = 0.5 * np.add.reduceat(c_hat.astype(np.float64), h["off"][:-1])
        s.update(p_hat=_up(p_hat), c_hat=_up(c_hat), budget=_up(budget.astype(np.float32)))
        return s
    if kind == "fixed":
        s["target"] = _up(_targets(h))
        return s
    s["p"] = _up(h["p"])
    if kind == "replicates":
        return s
    s["rewards"] = _up(h["rewards"])
    if kind in ("logged", "mean"):
        mask, pi = _logged(case, h)
        if kind == "logged":
            s.update(mask=_up(mask), pi=_up(pi))
        else:
            mean = np.add.reduceat(h["rewards"].astype(np.float64), h["off"][:-1]) / h["sizes"]
            c = mask * (h["rewards"] - mean[h["owner"]]) / h["sizes"][h["owner"]]
            s["coeff"] = _up(c.astype(np.float32))
    s["scores"] = _scores(case, h["nv"], seed)
    # A program keeps the audits' workspace from one call to the next.
    need = 0
    if kind == "audit":
        need = pair.pair_audit_workspace_bytes(B, case["gmax"], case["D"], case["R"])
    elif kind == "direction":
        need = pair.pair_audit_direction_workspace_bytes(B, case["gmax"], case["D"], case["R"])
    elif kind == "exact":
        need = pair.pair_audit_exact_workspace_bytes(B, case["gmax"], case["D"])
    if need:
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


def _targets(h):
    """First-order targets of the fixed-size design: uniform on [0.08, 0.92],
    scaled to the nearest admissible integer sum, all below 0.97."""
    t = h["rng"].uniform(0.08, 0.92, h["nv"])
    for b in range(h["sizes"].size):
        lo, hi = int(h["off"][b]), int(h["off"][b + 1])
        g = hi - lo
        x = t[lo:hi]
        while True:
            n = int(min(max(round(x.sum()), 1), g - 1))
            y = x * (n / x.sum())
            if y.max() < 0.97:
                break
            x = h["rng"].uniform(0.08, 0.92, g)
        t[lo:hi] = y
    return t.astype(np.float32)


# --------------------------------------------------------------------- run --
def run(s):
    case, kind, gmax, nv = s["case"], s["kind"], s["gmax"], s["nv"]
    if kind == "step":
        a = pair.design_coeffs(s["off"], s["p"], s["rewards"], s["seed"], 3, gmax, nv=nv)
        g = pair.weighted_grad(s["off"], s["scores"], a["coeff"], nv=nv)
        return {"design": a, "grad": g}
    if kind == "logged":
        c = pair.edge_coeffs(s["off"], s["rewards"], s["mask"], s["pi"], gmax, nv=nv,
                             rule=RULES[case["rule"]], wmax=WMAX)
        g = pair.weighted_grad(s["off"], s["scores"], c["coeff"], nv=nv)
        return {"fold": c, "grad": g}
    if kind == "mean":
        return pair.weighted_grad(s["off"], s["scores"], s["coeff"], nv=nv, reduce=True)
    if kind == "replicates":
        return pair.design_inclusion(s["off"], s["p"], s["seed"], 0, case["R"], gmax, nv=nv)
    if kind == "audit":
        return pair.audit(s["off"], s["scores"], s["rewards"], s["p"], s["seed"], 0, case["R"],
                          gmax, nv=nv, workspace=s["ws"], rule=RULES[case["rule"]], wmax=WMAX)
    if kind == "direction":
        return pair.audit_direction(s["off"], s["scores"], s["rewards"], s["p"], s["seed"], 0,
                                    case["R"], gmax, rule=RULES[case["rule"]], wmax=WMAX, nv=nv,
                                    workspace=s["ws"])
    if kind == "exact":
        return pair.audit_exact(s["off"], s["scores"], s["rewards"], s["p"], gmax,
                                rule=RULES[case["rule"]], wmax=WMAX, want_gram=True, nv=nv,
                                workspace=s["ws"])
    if kind == "alloc":
        # The step needs the probabilities and logs the objective; it asks for
        # no solver diagnostics.
        pi = torch.empty(nv, dtype=torch.float32, device=DEV)
        obj = torch.empty(s["B"], dtype=torch.float64, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        pair.pair_design_alloc(s["B"], nv, gmax, s["off"], s["p_hat"], s["c_hat"], None,
                               s["budget"], PI_MIN, pair.DESIGN_PAIR, pi, objective=obj,
                               d_status=status)
        return {"pi": pi, "objective": obj, "status": status}
    f = pair.cps_fit(s["off"], s["target"], gmax, nv=nv)
    d = pair.cps_draw(s["off"], f["w"], f["n"], s["seed"], 0, case["R"], gmax, nv=nv)
    return {"fit": f, "draw": d}


# -------------------------------------------------------------------- work --
def _live_share(case):
    """Expected share of prompts whose rewards are not all equal."""
    if case["gmin"] != case["gmax"]:
        return 1.0
    g = case["gmax"]   # 2 B(g + 1/2, 1/2) / B(1/2, 1/2): all succeed or all fail
    return 1.0 - 2.0 * math.exp(math.lgamma(g + 0.5) - math.lgamma(0.5) - math.lgamma(g + 1.0))


def work(case):
    """Bytes: inputs that the result depends on, once (score rows of drawn
    rollouts in prompts with unequal rewards), and outputs once.  Flops: the
    products with the score rows; for the audits one Gram matrix per prompt
    and one quadratic form per replicate, the least that gives the result."""
    kind, B, gmax = case["kind"], case["B"], case["gmax"]
    sizes = _sizes(case).astype(np.float64)
    nv, g2 = float(sizes.sum()), float((sizes * (sizes + 1)).sum())
    R, D = case.get("R", 1), case.get("D", 0)
    elt = 4 if case.get("dtype") == "f32" else 2
    small = 8.0 * (B + 1) + 8.0 * nv
    if kind in ("step", "logged", "mean"):
        rows = 0.55 * nv * _live_share(case)
        out = D * 4.0 * (1 if kind == "mean" else B)
        extra = 4.0 * B * gmax * gmax if kind != "mean" else 0.0
        return {"bytes": rows * D * elt + out + small + extra, "flops": 2.0 * rows * D}
    if kind == "replicates":
        return {"bytes": R * nv + 8.0 * R * B + 4.0 * B * gmax * gmax + small, "flops": 0.0}
    if kind in ("audit", "direction"):
        live = _live_share(case)
        out = 8.0 * B * R if kind == "audit" else 0.0
        return {"bytes": live * nv * D * 2 + out + small, "flops": live * g2 * (D + R)}
    if kind == "exact":
        return {"bytes": nv * D * 2 + 8.0 * B * gmax * gmax + small, "flops": g2 * D}
    if kind == "alloc":
        return {"bytes": 16.0 * nv + 16.0 * B, "flops": 8.0 * g2}
    return {"bytes": 24.0 * nv + 4.0 * B * gmax * gmax + R * nv + 4.0 * R * B,
            "flops": 4.0 * float((sizes ** 3).sum())}


# --------------------------------------------------------------- tolerance --
def tolerance(case):
    kind = case["kind"]
    if kind == "replicates":
        return {"rel": 1e-7, "max": 1e-6}
    if kind == "audit":
        # one fp16 rounding of the replicate coefficients: 1e-4 .. 5e-4 seen
        # against 64 bits
        return {"rel": 2e-3, "max": 2e-2}
    if kind == "alloc":
        return {"rel": 1e-6, "max": 1e-5}   # fp32 probabilities, converged to 1e-13
    if kind == "fixed":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.002}   # odds fitted to 1e-12
    # fp32 sums and coefficients: 1e-7 .. 3e-7 seen against 64 bits
    return {"rel": 2e-6, "max": 1e-4}


# ------------------------------------------------------- 64-bit references --
_M32 = 0xFFFFFFFF


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _mulhilo(m, c):
    m0, m1 = m & _M32, m >> 32
    c0, c1 = c & _M32, (c >> 32) & _M32
    p00 = c0 * m0
    p01 = c0 * m1 + ((p00 >> 32) & _M32)
    p10 = c1 * m0 + (p01 & _M32)
    hi = c1 * m1 + ((p01 >> 32) & _M32) + ((p10 >> 32) & _M32)
    return hi, (p10 << 32) | (p00 & _M32)


def _uniforms(seed, rep0, R, B, gmax):
    """[R][B][4 * blocks] top 32 bits of Philox4x64-10 at counter (replicate,
    prompt, vertex // 4, 0), key (seed, 0)."""
    nb = (gmax + 3) // 4
    shape = (R, B, nb)
    c0 = (torch.arange(R, device=DEV) + rep0).view(R, 1, 1).expand(shape).clone()
    c1 = torch.arange(B, device=DEV).view(1, B, 1).expand(shape).clone()
    c2 = torch.arange(nb, device=DEV).view(1, 1, nb).expand(shape).clone()
    c3 = torch.zeros_like(c2)
    k0, k1 = seed & ((1 << 64) - 1), 0
    for r in range(10):
        if r:
            k0 += 0x9E3779B97F4A7C15
            k1 += 0xBB67AE8584CAA73B
        h0, l0 = _mulhilo(0xD2E7470EE14C6C93, c0)
        h1, l1 = _mulhilo(0xCA5A826395121157, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ _signed(k0), l1, h0 ^ c3 ^ _signed(k1), l0
    return torch.stack([(x >> 32) & _M32 for x in (c0, c1, c2, c3)], dim=-1).view(R, B, 4 * nb)


def _padded(h, x, gmax, fill=0.0):
    out = np.full((h["sizes"].size, gmax), fill, dtype=np.float64)
    out[h["owner"], np.arange(h["nv"]) - h["off"][:-1][h["owner"]]] = x
    return torch.from_numpy(out).to(DEV)


def _indicators(case, h, seed, rep0, R):
    """[R][B][gmax] in {0, 1} as fp64."""
    gmax = case["gmax"]
    p = _padded(h, h["p"], gmax)
    u = _uniforms(seed, rep0, R, case["B"], gmax)[:, :, :gmax]
    return (u < torch.floor(p * 4294967296.0).to(torch.int64)[None]).double()


def _fold(rule, J, r, p, rho, g):
    """Coefficients [..., G] of indicators J [..., G] for one prompt, uncentred
    (the centred rules' coefficients sum to zero in exact arithmetic)."""
    n = r.numel()
    dr = r[:, None] - r[None, :]
    eye = torch.eye(n, dtype=torch.float64, device=DEV)
    w = torch.where(eye > 0, torch.zeros_like(rho), 1.0 / rho)
    if rule in ("unweighted", "ratio_ke"):
        w = 1.0 - eye
    elif rule == "clipped":
        w = w.clamp(max=WMAX)
    elif rule == "marginal":
        w = (1.0 - eye) / p[:, None]
    c = J * (J @ (w * dr).T)
    k = J.sum(-1, keepdim=True)
    den = torch.full_like(k, float(g * (g - 1)))
    if rule == "ratio_ke":
        den = k * (k - 1)
    elif rule == "selfnorm":
        den = (J * (J @ w.T)).sum(-1, keepdim=True)
    return torch.where(k >= 2, c / den, torch.zeros_like(c))


def _prompt(h, b):
    lo, hi = int(h["off"][b]), int(h["off"][b + 1])
    r = torch.from_numpy(h["rewards"][lo:hi].astype(np.float64)).to(DEV)
    p32 = torch.from_numpy(h["p"][lo:hi]).to(DEV)
    rho = (p32[:, None] * p32[None, :]).double()   # the logged fp32 product
    return lo, hi, r, p32.double(), rho


def _exact_grad(case, h, seed, coeffs):
    """Per-prompt gradients in fp64 from per-prompt coefficient vectors."""
    S = _scores(case, h["nv"], seed)
    out = torch.empty((case["B"], case["D"]), dtype=torch.float64, device=DEV)
    for b, c in enumerate(coeffs):
        lo, hi = int(h["off"][b]), int(h["off"][b + 1])
        out[b] = c @ S[lo:hi].double()
    return out


def _exact_steps(case, seed):
    h = _host(case, seed)
    kind, B = case["kind"], case["B"]
    if kind == "logged":
        mask, _ = _logged(case, h)
        J = _padded(h, mask, case["gmax"])
    else:
        J = _indicators(case, h, seed, 3, 1)[0]
    rule = case.get("rule", "ht")
    coeffs, ess, mw = [], [], []
    pi = torch.zeros((B, case["gmax"], case["gmax"]), dtype=torch.float64, device=DEV)
    for b in range(B):
        lo, hi, r, p, rho = _prompt(h, b)
        g = hi - lo
        j = J[b, :g]
        coeffs.append(_fold(rule, j, r, p, rho, g))
        pi[b, :g, :g] = p[:, None] * p[None, :] * (1 - torch.eye(g, device=DEV)) + torch.diag(p)
        if kind == "logged":
            w = 1.0 / rho
            if rule in ("unweighted", "ratio_ke"):
                w = torch.ones_like(rho)
            elif rule == "clipped":
                w = w.clamp(max=WMAX)
            elif rule == "marginal":
                w = 0.5 * (1.0 / p[:, None] + 1.0 / p[None, :])
            w = torch.triu(w * j[:, None] * j[None, :], 1)
            ess.append(w.sum() ** 2 / (w * w).sum() if float(j.sum()) >= 2 else w.sum())
            mw.append(w.max())
    out = _exact_grad(case, h, seed, coeffs)
    coeff = torch.cat(coeffs)
    if kind == "step":
        return {"design": {"coeff": coeff, "pi": pi}, "grad": {"out": out}}
    return {"fold": {"coeff": coeff, "ess": torch.stack(ess), "max_weight": torch.stack(mw)},
            "grad": {"out": out}}


def _exact_mean(case, seed):
    s = prepare(case, seed)
    out = torch.zeros(case["D"], dtype=torch.float64, device=DEV)
    for lo in range(0, s["nv"], 256):
        out += s["coeff"][lo:lo + 256].double() @ s["scores"][lo:lo + 256].double()
    return {"out": out / case["B"]}


def _exact_mc(case, seed):
    """The audits straight from their definition: every replicate's estimate
    minus the target, its square summed over the score columns in chunks."""
    h = _host(case, seed)
    S = _scores(case, h["nv"], seed)
    R, D, B, direction = case["R"], case["D"], case["B"], case["kind"] == "direction"
    J = _indicators(case, h, seed, 0, R)
    e = torch.zeros((B, R), dtype=torch.float64, device=DEV)
    first = torch.zeros(B, dtype=torch.float64, device=DEV)
    second = torch.zeros(B, dtype=torch.float64, device=DEV)
    cols = max(512, (1 << 27) // R)
    for b in range(B):
        lo, hi, r, p, rho = _prompt(h, b)
        g = hi - lo
        u = _fold(case["rule"], J[:, b, :g], r, p, rho, g)
        a = (r - r.mean()) / (g - 1)
        dot = torch.zeros(R, dtype=torch.float64, device=DEV)
        sq, tt, bias = torch.zeros_like(dot), 0.0, 0.0
        for c in range(0, D, cols):
            s = S[lo:hi, c:c + cols].double()
            t = a @ s
            y = u @ s
            if direction:
                dot += y @ t
                sq += (y * y).sum(1)
                tt = tt + t @ t
            else:
                sq += ((y - t) ** 2).sum(1)
                bias = bias + ((y.mean(0) - t) ** 2).sum()
        if direction:
            ok = (sq > 0) & (tt > 0)
            den = torch.sqrt(torch.where(ok, sq * tt, torch.ones_like(sq)))
            first[b] = torch.where(ok, dot / den, torch.zeros_like(dot)).mean()
            second[b] = torch.sqrt(tt)
        elif float((r - r[0]).abs().max()) > 0:
            e[b], first[b], second[b] = sq, sq.mean(), torch.sqrt(bias)
    if direction:
        return {"cosine": first, "target_norm": second}
    return {"mse": first, "bias_norm": second, "rep_sqerr": e}


def _exact_closed(case, seed):
    """Prop. 1 from the Gram matrix in fp64: the shared-vertex term of vertex i
    is |sum_j p_j v_ij|^2 - sum_j p_j^2 |v_ij|^2."""
    h = _host(case, seed)
    S = _scores(case, h["nv"], seed)
    B, gm = case["B"], case["gmax"]
    gram = torch.zeros((B, gm, gm), dtype=torch.float64, device=DEV)
    mse = torch.zeros(B, dtype=torch.float64, device=DEV)
    bias = torch.zeros_like(mse)
    for b in range(B):
        lo, hi, r, p, rho = _prompt(h, b)
        g = hi - lo
        s = S[lo:hi].double()
        K = s @ s.T
        gram[b, :g, :g] = K
        off = 1.0 - torch.eye(g, dtype=torch.float64, device=DEV)
        w = 1.0 / rho
        if case["rule"] == "unweighted":
            w = torch.ones_like(rho)
        elif case["rule"] == "clipped":
            w = w.clamp(max=WMAX)
        elif case["rule"] == "marginal":
            w = (1.0 / p)[:, None].expand(g, g)
        dr = r[:, None] - r[None, :]
        A = 0.5 * dr * w * off
        C = A.T                                    # v_ij = A_ij s_i + C_ij s_j
        M = 0.5 * g * (g - 1)
        beta = ((p[:, None] * p[None, :] * A - 0.5 * dr) * off).sum(1) / M
        kd = torch.diag(K)
        v2 = A * A * kd[:, None] + 2 * A * C * K + C * C * kd[None, :]
        rr = p[:, None] * p[None, :]
        tr = 0.5 * (rr * (1 - rr) * v2 * off).sum()
        X = p[None, :] * C * off + torch.diag((p[None, :] * A * off).sum(1))
        shared = ((X @ K) * X).sum(1) - (p[None, :] ** 2 * v2 * off).sum(1)
        tr = tr + (p * (1 - p) * shared).sum()
        b2 = (beta @ K @ beta).clamp(min=0.0)
        bias[b], mse[b] = torch.sqrt(b2), b2 + tr / (M * M)
    return {"gram": gram, "mse": mse, "bias_norm": bias}


def _exact_alloc(case, seed):
    """Coordinate minimisation for a multiplier, the multiplier by bisection,
    all prompts at once in fp64."""
    s = prepare(case, seed)
    h = _host(case, seed)
    g = case["gmax"]
    ph, ch = (_padded(h, s[k].cpu().numpy(), g).cpu().numpy() for k in ("p_hat", "c_hat"))
    valid = _padded(h, np.ones(h["nv"]), g).cpu().numpy() > 0
    bud, pmin = s["budget"].double().cpu().numpy(), float(np.float32(PI_MIN))
    a = ph[:, :, None] * (1 - ph[:, None, :]) + (1 - ph[:, :, None]) * ph[:, None, :]
    a *= valid[:, :, None] & valid[:, None, :]
    d = np.arange(g)
    a[:, d, d] = 0.0
    bv = np.maximum(np.sqrt(a).sum(2) ** 2 - a.sum(2), 0.0)
    c = np.where(valid, ch, 1.0)

    def solve(lam, pi):
        for _ in range(400):
            old = pi.copy()
            for i in range(g):
                A = (a[:, i, :] / pi).sum(1) + bv[:, i]
                pi[:, i] = np.where(valid[:, i], np.clip(np.sqrt(A / (lam * c[:, i])), pmin, 1.0),
                                    1.0)
            if np.abs(pi / old - 1).max() < 1e-14:
                break
        return pi, (c * pi * valid).sum(1)

    lo, hi = np.full(case["B"], -40.0), np.full(case["B"], 20.0)
    pi = np.ones((case["B"], g))
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        pi, spent = solve(np.exp(mid), pi)
        lo, hi = np.where(spent > bud, mid, lo), np.where(spent > bud, hi, mid)
    phi = 0.5 * (a / (pi[:, :, None] * pi[:, None, :])).sum((1, 2)) + (bv / pi).sum(1)
    return {"pi": torch.from_numpy(pi[valid]), "objective": torch.from_numpy(phi)}


def _pair_probs(w, n, valid, chunk=32):
    """First-order and joint probabilities of the fixed-size design from the
    elementary symmetric polynomials without each pair of units."""
    B, g = w.shape
    pi = torch.zeros((B, g, g), dtype=torch.float64, device=DEV)
    for lo in range(0, B, chunk):
        ww, vv, nn = w[lo:lo + chunk], valid[lo:lo + chunk], n[lo:lo + chunk]
        m = ww.shape[0]
        full = torch.zeros((m, g + 1), dtype=torch.float64, device=DEV)
        full[:, 0] = 1.0
        E = torch.zeros((m, g, g, g + 1), dtype=torch.float64, device=DEV)
        E[..., 0] = 1.0
        for u in range(g):
            x = (ww[:, u] * vv[:, u])[:, None]
            full[:, 1:] = full[:, 1:] + x * full[:, :-1]
            keep = torch.ones((g, g), dtype=torch.float64, device=DEV)
            keep[u, :] = 0.0
            keep[:, u] = 0.0
            E[..., 1:] = E[..., 1:] + (x[:, :, None] * keep[None])[..., None] * E[..., :-1]
        en = full.gather(1, nn[:, None])[:, :, None]
        i1 = (nn - 1)[:, None, None, None].expand(m, g, g, 1)
        i2 = (nn - 2).clamp(min=0)[:, None, None, None].expand(m, g, g, 1)
        one = torch.diagonal(E.gather(3, i1)[..., 0], dim1=1, dim2=2) * ww / en[:, :, 0]
        two = E.gather(3, i2)[..., 0] * ww[:, :, None] * ww[:, None, :] / en
        two = two * (nn >= 2)[:, None, None]
        eye = torch.eye(g, dtype=torch.float64, device=DEV)[None]
        pi[lo:lo + chunk] = (two * (1 - eye) + one[:, :, None] * eye) * \
            (vv[:, :, None] * vv[:, None, :])
    return pi


def _exact_fixed(case, seed):
    """Odds by Newton's method on the log-odds (the Hessian is the design's
    covariance), joint probabilities without each pair."""
    s = prepare(case, seed)
    h = _host(case, seed)
    g = case["gmax"]
    t = _padded(h, s["target"].double().cpu().numpy(), g, 0.5)
    valid = _padded(h, np.ones(h["nv"]), g)
    sums = (t * valid).sum(1)
    n = torch.round(sums).to(torch.int64)
    t = t * (n / sums)[:, None]
    size = valid.sum(1, keepdim=True)
    th = torch.log(t / (1 - t)) * valid
    th = (th - th.sum(1, keepdim=True) / size) * valid
    eye = torch.eye(g, dtype=torch.float64, device=DEV)[None]
    for _ in range(12):
        joint = _pair_probs(torch.exp(th), n, valid)
        pi = torch.diagonal(joint, dim1=1, dim2=2)
        H = joint - pi[:, :, None] * pi[:, None, :]
        H = H + valid[:, :, None] * valid[:, None, :] / size[:, :, None] + \
            eye * (1 - valid)[:, :, None]
        d = torch.linalg.solve(H.cpu(), ((t - pi) * valid).cpu()[:, :, None])[:, :, 0].to(DEV)
        d = d * valid
        d = d * (1.0 / d.abs().amax(1, keepdim=True).clamp(min=1.0))
        th = th + d
        th = (th - th.sum(1, keepdim=True) / size) * valid
    w = torch.exp(th)
    return {"fit": {"w": w[valid > 0], "pi_joint": _pair_probs(w, n, valid)}}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "logged"):
        return _exact_steps(case, seed)
    if kind == "mean":
        return _exact_mean(case, seed)
    if kind == "replicates":
        h = _host(case, seed)
        p = _padded(h, h["p"], case["gmax"])
        eye = torch.eye(case["gmax"], dtype=torch.float64, device=DEV)[None]
        return {"pi": p[:, :, None] * p[:, None, :] * (1 - eye) + p[:, :, None] * eye}
    if kind in ("audit", "direction"):
        return _exact_mc(case, seed)
    if kind == "exact":
        return _exact_closed(case, seed)
    return _exact_alloc(case, seed) if kind == "alloc" else _exact_fixed(case, seed)
