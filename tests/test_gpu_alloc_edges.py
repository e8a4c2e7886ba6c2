"""The allocation sweep where it can go wrong: one vertex, two, both ends of
the wave, floors near 0 (the state is 1 / pi), vertices without contrast
(predictions 0 and 1: A = 0), costs over twelve decades, score norms.

Bar: the oracle's own KKT checker at the returned fp32 probabilities, whose
rounding moves a gradient A / pi^2 by up to 3 * 2^-24 relative and the spent
budget by 2^-24: 1e-6, four times their sum, for sound inputs."""
import numpy as np
import pytest
import torch

import paper_2608_11368_amd as pair
from oracle import alloc
from tests.gpu_util import DEV, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pi_min", [0.08, 1e-6])
@pytest.mark.parametrize("kind", ["plain", "scaled", "costs", "certain", "pointwise"])
def test_kkt_at_the_edges(kind, pi_min):
    sizes = [1, 2, 3, 15, 16, 17, 31, 33, 63, 64]
    rng = np.random.default_rng(len(kind))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    nv = int(off[-1])
    p = rng.uniform(0.02, 0.98, nv).astype(np.float32)
    if kind == "certain":
        p[rng.random(nv) < 0.5] = 0.0
        p[rng.random(nv) < 0.3] = 1.0
    c = rng.lognormal(8.0, 1.0, nv)
    if kind == "costs":
        c = 10.0 ** rng.uniform(-6.0, 6.0, nv)
    c = c.astype(np.float32)
    m = rng.uniform(0.1, 3.0, nv).astype(np.float32) if kind == "scaled" else None
    bud = (0.5 * np.add.reduceat(c.astype(np.float64), off[:-1])).astype(np.float32)
    t = lambda a: None if a is None else torch.from_numpy(a).to(DEV)
    design = pair.DESIGN_POINTWISE if kind == "pointwise" else pair.DESIGN_PAIR
    got = pair.design_alloc(t(off), t(p), t(c), t(bud), 64, pi_min=pi_min, design=design, m_hat=t(m))
    torch.cuda.synchronize()
    pi, iters = got["pi"].cpu().numpy().astype(np.float64), got["iters"].cpu().numpy()
    obj = got["objective"].cpu().numpy()
    assert int(got["status"].item()) == 0 and np.all(iters >= 0)
    floor = float(np.float32(pi_min))
    worst = 0.0
    for b in range(len(sizes)):
        s = slice(off[b], off[b + 1])
        pv, cv, x = p[s].astype(np.float64), c[s].astype(np.float64), pi[s]
        assert np.all(x >= floor) and np.all(x <= 1.0)
        a = alloc.edge_proxy(pv, None if m is None else m[s].astype(np.float64))
        bv = alloc.vertex_term(a)
        want = alloc.objective_pi(x, a, bv)
        # the objective is taken at the fp64 probabilities: 2^-23 from these
        assert abs(obj[b] - want) <= 2.0 ** -22 * max(want, 1e-300), (b, obj[b], want)
        if kind == "pointwise":
            a, bv = np.zeros_like(a), pv * (1.0 - pv)
        if not np.any(bv > 0.0):
            if not np.any(a > 0.0):
                continue   # no contrast at all: any design is optimal
        kk = alloc.kkt_residual(x, a, bv, cv, float(bud[b]), floor)[0]
        # An optimum without contrast at some vertices may leave budget unspent.
        worst = max(worst, kk if cv @ x > 0.999 * bud[b] else 0.0)
        assert cv @ x <= float(bud[b]) * (1.0 + 2.0 ** -22)
    log(f"alloc edges {kind} pi_min={pi_min}: worst KKT {worst:.2e}, sweeps max {iters.max()}")
    assert worst <= 1e-6
