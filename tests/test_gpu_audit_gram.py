"""The audit's Gram path where it can go wrong: group sizes at the edges of
the 16-row blocks, score widths at the edges of chunks and slices, ragged
batches that mix the shapes, replicate counts that leave workgroups without
a slice, and rows whose fp32 products would overflow, vanish or nearly cancel.

Bound: K_ij has exact products and fp32 runs of a few dozen sums, and the
fold's fp32 coefficients carry a few roundings, so |Delta e_r| is a small
multiple c of 2^-24 times A_r^2 with A_r = sum_i (|u_ri| + |a_i|) |s_i|, the size
of what cancels in delta_r S.  c = 4 is used; the reference is the fp64
oracle's explicit edge sum."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11368_amd as pair
import workloads as wl
from tests.gpu_util import DEV, log, scores_to_host

pytestmark = pytest.mark.gpu

C = 4 * 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pair.lib()


def _case(sizes, D, kind, seed):
    rng = np.random.default_rng(seed)
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    nv = int(off[-1])
    rewards = rng.random(nv).astype(np.float32)
    p = rng.uniform(0.2, 1.0, nv).astype(np.float32)
    ld = (D + 7) // 8 * 8
    x = np.full((nv, ld), np.nan, dtype=np.float32)
    x[:, :D] = rng.standard_normal((nv, D))
    if kind == "huge":
        x[::2, :D] *= np.float32(2.0 ** 58)
    elif kind == "tiny":
        x[:, :D] *= np.float32(2.0 ** -60)
    elif kind == "mixed":
        x[::3, :D] *= np.float32(2.0 ** -100)
        x[1::3, :D] *= np.float32(2.0 ** 40)
    elif kind == "zero_rows":
        x[::2, :D] = 0.0
    elif kind == "common":
        x[:, :D] += 300.0 * rng.standard_normal(D).astype(np.float32)
    s = torch.from_numpy(x).to(torch.bfloat16)
    return off, rewards, p, s, int(max(sizes))


@pytest.mark.parametrize("sizes,D,R,kind", [
    ([2, 15, 16], 1, 5, "normal"), ([16, 3], 511, 65, "normal"), ([16], 512, 600, "normal"),
    ([17, 2, 16], 513, 64, "normal"), ([32, 31], 2047, 40, "normal"), ([33, 16], 2048, 40, "normal"),
    ([48, 5, 17, 33], 2049, 70, "normal"), ([49, 16, 32, 48], 4225, 33, "normal"),
    ([64, 2, 63], 6145, 300, "normal"), ([16, 16], 8193, 20, "normal"), ([16, 9], 1100, 40, "huge"),
    ([64, 20], 300, 40, "huge"), ([16, 40], 900, 40, "tiny"), ([16, 64, 31], 2100, 40, "mixed"),
    ([16, 33], 700, 40, "zero_rows"), ([16, 50], 3000, 40, "common")])
def test_audit_against_oracle(sizes, D, R, kind):
    off, rewards, p, s, gmax = _case(sizes, D, kind, 17 * D + R)
    log(f"audit gram {kind} sizes={sizes} D={D} R={R}")
    nv, B = int(off[-1]), len(sizes)
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    sd = s.to(DEV)[:, :D]
    got = pair.audit(dev[0], sd, dev[1], dev[2], 99, 7, R, gmax, nv=nv)
    torch.cuda.synchronize()
    assert int(got["status"].item()) == 0
    host = scores_to_host(s)[:, :D]
    want = oracle.audit(off, host, rewards, p, 99, 7, R, gmax=gmax)
    assert np.array_equal(got["edge_count"].cpu().numpy(), want["edge_count"])
    d = oracle.design_inclusion(off, p, 99, 7, R, gmax)
    full, _ = oracle.pair_coeffs(off, rewards)
    norms = np.sqrt((s[:, :D].double().numpy() ** 2).sum(1))
    A = np.zeros((B, R))
    for r in range(R):
        u, _ = oracle.pair_coeffs(off, rewards, d["mask"][r], d["pi"])
        A[:, r] = np.add.reduceat((np.abs(u) + np.abs(full)) * norms, off[:-1])
    e = got["rep_sqerr"].cpu().numpy().astype(np.float64)
    worst = np.max(np.abs(e - want["rep_sqerr"]) / (C * A ** 2 + 2.0 ** -24 * want["rep_sqerr"]))
    mse = got["mse"].cpu().numpy()
    m = np.max(np.abs(mse - want["mse"]) / (C * (A ** 2).mean(1)))
    # the bias is linear in the coefficients, also where the rows nearly cancel
    bias = got["bias_norm"].cpu().numpy()
    bb = np.max(np.abs(bias - want["bias_norm"]) / (C * A.mean(1)))
    log(f"  in units of the bound: e {worst:.3f}, mse {m:.3f}, bias {bb:.3f}")
    assert worst <= 1.0 and m <= 1.0 and bb <= 1.0


RULES = [pair.RULE_HT, pair.RULE_UNWEIGHTED, pair.RULE_RATIO_KE, pair.RULE_CLIPPED,
         pair.RULE_SELFNORM, pair.RULE_MARGINAL]


@pytest.mark.parametrize("logged", [False, True])
@pytest.mark.parametrize("rule", RULES)
def test_rules_against_oracle(rule, logged):
    """Every rule's fold, normaliser and centring, from p and from a logged rho
    block, over group sizes on both sides of the 16-row blocks, to the same
    bound; the logged weights span a decade, so the fold's terms exceed its sum:
    A_r has the sum of their sizes over the normaliser."""
    sizes, D, R, wmax = [2, 5, 16, 17, 33, 48, 64], 700, 130, 3.0
    off, rewards, p, s, gmax = _case(sizes, D, "normal", 50 + rule)
    B, nv = len(sizes), int(off[-1])
    pi_w = None
    if logged:
        pi_w = np.random.default_rng(rule).uniform(0.1, 1.0, (B, gmax, gmax)).astype(np.float32)
    log(f"audit gram rule {rule} logged={logged}")
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    got = pair.audit(dev[0], s.to(DEV)[:, :D], dev[1], dev[2], 77, 1, R, gmax, nv=nv, rule=rule,
                     wmax=wmax, pi_w=None if pi_w is None else torch.from_numpy(pi_w).to(DEV))
    torch.cuda.synchronize()
    assert int(got["status"].item()) == 0
    want = oracle.audit(off, scores_to_host(s)[:, :D], rewards, p, 77, 1, R, gmax=gmax, rule=rule,
                        wmax=wmax, pi_w=pi_w)
    assert np.array_equal(got["edge_count"].cpu().numpy(), want["edge_count"])
    d = oracle.design_inclusion(off, p, 77, 1, R, gmax)
    rho = d["pi"] if pi_w is None else pi_w
    full, _ = oracle.pair_coeffs(off, rewards)
    norms = np.sqrt((s[:, :D].double().numpy() ** 2).sum(1))
    e = got["rep_sqerr"].cpu().numpy().astype(np.float64)
    mse, bias = got["mse"].cpu().numpy(), got["bias_norm"].cpu().numpy()
    top = np.zeros(3)
    for b in range(B):
        lo, hi = int(off[b]), int(off[b + 1])
        g = hi - lo
        blk = np.triu(rho[b, :g, :g].astype(np.float64), 1)
        blk = blk + blk.T + np.eye(g)
        mar = np.diag(rho[b, :g, :g]).astype(np.float64)
        w = 1.0 / blk
        if rule in (pair.RULE_UNWEIGHTED, pair.RULE_RATIO_KE):
            w = np.ones((g, g))
        elif rule == pair.RULE_CLIPPED:
            w = np.minimum(w, wmax)
        elif rule == pair.RULE_MARGINAL:
            w = np.repeat(1.0 / mar[:, None], g, axis=1)
        size = w * np.abs(rewards[lo:hi, None].astype(np.float64) - rewards[None, lo:hi])
        J = d["mask"][:, lo:hi].astype(np.float64)
        k = J.sum(1)
        den = np.full(R, g * (g - 1.0))
        if rule == pair.RULE_RATIO_KE:
            den = k * (k - 1)
        elif rule == pair.RULE_SELFNORM:
            den = np.einsum("ri,ij,rj->r", J, w - np.diag(np.diag(w)), J)
        fold = J * (J @ size.T) / np.where(k >= 2, den, np.inf)[:, None]
        A = ((fold + np.abs(full[lo:hi])) * norms[lo:hi]).sum(1)
        top = np.maximum(top, [
            np.max(np.abs(e[b] - want["rep_sqerr"][b]) / (C * A ** 2 + 2.0 ** -24 * want["rep_sqerr"][b])),
            abs(mse[b] - want["mse"][b]) / (C * (A ** 2).mean()),
            abs(bias[b] - want["bias_norm"][b]) / (C * A.mean())])
    log(f"  in units of the bound: e {top[0]:.3f}, mse {top[1]:.3f}, bias {top[2]:.3f}")
    assert np.all(top <= 1.0)


@pytest.mark.parametrize("R", [1, 255, 256, 257, 2100])
def test_replicates_past_the_slices_are_drawn(R):
    """One slice per prompt and more replicates than its workgroup draws:
    bitwise the e_r and edge counts of a call per replicate range."""
    off, rewards, p, s, gmax = _case([16, 40, 7], 96, "normal", R)
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    sd, nv = s.to(DEV), int(off[-1])
    one = pair.audit(dev[0], sd, dev[1], dev[2], 5, 3, R, gmax, nv=nv)
    cut = (R + 1) // 2
    parts = [pair.audit(dev[0], sd, dev[1], dev[2], 5, 3 + lo, hi - lo, gmax, nv=nv)
             for lo, hi in ((0, cut), (cut, R)) if hi > lo]
    for key in ("rep_sqerr", "edge_count"):
        assert torch.equal(torch.cat([x[key] for x in parts], dim=1), one[key])


@pytest.mark.parametrize("sizes,D", [([64, 33], 1 << 20), ([48, 50], (1 << 21) + 2056)])
def test_long_rows_are_summed_in_short_runs(sizes, D):
    """Rows far longer than 128 slices of 2048 columns, with a component ten
    times the rest in common: K's fp32 runs are 128 columns each, so their
    roundings are N = D / 128 independent ones of 2^-24 at most, and e_r and
    |t|^2 are within 2^-24 / sqrt(N) of A^2, what cancels in them (runs over a
    whole slice round with a bias instead: 1.1 to 2.8 times this bound, now 0.07 to
    0.21 of it).  The fold's centring adds 2^-23 A_r |delta_r S| / sqrt(G)."""
    rng = np.random.default_rng(D)
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    nv, B, R, gmax = int(off[-1]), len(sizes), 20, max(sizes)
    rewards = rng.random(nv).astype(np.float32)
    p = rng.uniform(0.2, 1.0, nv).astype(np.float32)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(D)
    common = 10.0 * torch.randn(D, generator=gen, device=DEV)
    s = torch.empty((nv, D), dtype=torch.bfloat16, device=DEV)
    for i in range(nv):
        s[i] = (torch.randn(D, generator=gen, device=DEV) + common).to(torch.bfloat16)
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    log(f"audit gram long rows sizes={sizes} D={D}")
    got = pair.audit(dev[0], s, dev[1], dev[2], 9, 3, R, gmax, nv=nv)
    way = pair.audit_direction(dev[0], s, dev[1], dev[2], 9, 3, R, gmax, nv=nv)
    torch.cuda.synchronize()
    assert int(got["status"].item()) == 0 and int(way["status"].item()) == 0
    d = oracle.design_inclusion(off, p, 9, 3, R, gmax)
    full, _ = oracle.pair_coeffs(off, rewards)
    u = np.stack([oracle.pair_coeffs(off, rewards, d["mask"][r], d["pi"])[0] for r in range(R)])
    rows = torch.from_numpy(np.concatenate([u - full, full[None]])).to(DEV)
    eps = 2.0 ** -24 / np.sqrt(D / 128)
    for b in range(B):
        lo, hi = int(off[b]), int(off[b + 1])
        sq = torch.zeros(R + 1, dtype=torch.float64, device=DEV)
        norm = torch.zeros(hi - lo, dtype=torch.float64, device=DEV)
        for c in range(0, D, 1 << 16):
            x = s[lo:hi, c:c + (1 << 16)].double()
            sq += (rows[:, lo:hi] @ x).square().sum(1)
            norm += x.square().sum(1)
        sq, norm = sq.cpu().numpy(), norm.sqrt().cpu().numpy()
        A = ((np.abs(u) + np.abs(full))[:, lo:hi] * norm).sum(1)
        e = got["rep_sqerr"][b].double().cpu().numpy()
        worst = np.max(np.abs(e - sq[:R]) / (eps * A ** 2 + 2.0 ** -23 * A * np.sqrt(sq[:R] / (hi - lo))))
        At = (np.abs(full[lo:hi]) * norm).sum()
        t2 = float(way["target_norm"][b]) ** 2
        tn = abs(t2 - sq[R]) / (eps * At ** 2 + 2.0 ** -23 * At * np.sqrt(sq[R] / (hi - lo)))
        log(f"  in units of the bound: e {worst:.3f}, target {tn:.3f}")
        assert worst <= 1.0 and tn <= 1.0


@pytest.mark.parametrize("rule,R,c,D", [
    (pair.RULE_UNWEIGHTED, 200, 100.0, 4096), (pair.RULE_UNWEIGHTED, 200, 300.0, 70001),
    (pair.RULE_HT, 8, 300.0, 4096), (pair.RULE_HT, 8, 300.0, 70001)])
def test_bias_norm_with_a_common_component(rule, R, c, D):
    """Score rows that share a component c times the rest, except in the last
    prompt: |delta_bar S| cancels by about c sqrt(G).  Its error grows with the first
    power of that, as a sum per score column does: the coefficients carry
    a few roundings of 2^-24, so |Delta bias| <= 2^-23 A with A the mean over
    replicates of A_r (for the unweighted rule and rewards in {0, 1} the folds
    are whole numbers, and A is that of the target alone).  The quadratic form
    of K by itself misses this by up to 20."""
    rng = np.random.default_rng(int(c) + D)
    sizes = [16, 5, 64, 33, 20]
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    nv, gmax = int(off[-1]), 64
    whole = rule == pair.RULE_UNWEIGHTED
    rewards = (rng.permutation(nv) % 2 if whole else rng.random(nv)).astype(np.float32)
    p = rng.uniform(0.2, 1.0, nv).astype(np.float32)
    ld = (D + 7) // 8 * 8
    x = np.full((nv, ld), np.nan, dtype=np.float32)
    x[:, :D] = rng.standard_normal((nv, D))
    x[:off[-2], :D] += np.float32(c) * rng.standard_normal(D).astype(np.float32)
    s = torch.from_numpy(x).to(torch.bfloat16)
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    sd = s.to(DEV)[:, :D]
    log(f"audit bias, common component {c} D={D} R={R} rule={rule}")
    ws = torch.full((pair.pair_audit_workspace_bytes(len(sizes), gmax, D, R),), 255,
                    dtype=torch.uint8, device=DEV)
    got = [pair.audit(dev[0], sd, dev[1], dev[2], 3, 0, R, gmax, nv=nv, rule=rule, workspace=ws)
           for _ in range(2)]
    torch.cuda.synchronize()
    assert int(got[0]["status"].item()) == 0
    assert torch.equal(got[0]["bias_norm"], got[1]["bias_norm"])
    d = oracle.design_inclusion(off, p, 3, 0, R, gmax)
    full, _ = oracle.pair_coeffs(off, rewards)
    u = np.stack([oracle.pair_coeffs_rule(off, rewards, d["mask"][r], d["pi"], rule)["coeff"]
                  for r in range(R)])
    S = s[:, :D].double().numpy()
    norm = np.sqrt((S ** 2).sum(1))
    A = norm * (np.abs(full) + (0.0 if whole else np.abs(u).mean(0)))
    for b in range(len(sizes)):
        lo, hi = int(off[b]), int(off[b + 1])
        want = np.linalg.norm((u - full).mean(0)[lo:hi] @ S[lo:hi])
        unit = 2.0 ** -23 * A[lo:hi].sum()
        err = abs(float(got[0]["bias_norm"][b]) - want) / unit
        log(f"  G={hi - lo}: {err:.3f} of the bound, which is {unit / want:.1e} of the norm")
        assert err <= 1.0


def test_nonfinite_score_raises_in_any_slice():
    off, rewards, p, s, gmax = _case([16, 33], 5000, "normal", 4)
    dev = [torch.from_numpy(a).to(DEV) for a in (off, rewards, p)]
    for row, col, v in ((3, 4999, float("inf")), (20, 0, float("nan")), (48, 2500, float("-inf"))):
        bad = s.clone()
        bad[row, col] = v
        got = pair.audit(dev[0], bad.to(DEV), dev[1], dev[2], 5, 0, 20, gmax, nv=int(off[-1]))
        assert int(got["status"].item()) == pair.ST_NONFINITE
        other = 1 if row < 16 else 0
        ok = pair.audit(dev[0], s.to(DEV), dev[1], dev[2], 5, 0, 20, gmax, nv=int(off[-1]))
        assert torch.equal(got["rep_sqerr"][other], ok["rep_sqerr"][other])
