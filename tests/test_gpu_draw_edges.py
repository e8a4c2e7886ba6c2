"""Replicate draws where the work split can go wrong: group sizes around a
quad of four and around the whole wave, batches around a workgroup's prompts,
replicate counts around a workgroup's share.  Draws are bit-exact against the
oracle (integers and one fp32 product), so there is no tolerance."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11368_amd as pair
from tests.gpu_util import DEV, log

pytestmark = pytest.mark.gpu

SIZES = {"edges": [2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 61, 62, 63, 64], "one": [64],
         "twos": [2] * 33, "full": [64] * 16}


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _offsets(name):
    return np.concatenate([[0], np.cumsum(SIZES[name])]).astype(np.int64)


@pytest.mark.parametrize("name,R", [("edges", 1), ("edges", 2), ("edges", 15), ("edges", 16),
                                    ("edges", 17), ("edges", 300), ("one", 1), ("one", 65),
                                    ("twos", 7), ("twos", 64), ("full", 33)])
def test_design_draws(name, R):
    off = _offsets(name)
    nv, gmax, B = int(off[-1]), max(SIZES[name]), len(SIZES[name])
    rng = np.random.default_rng(R)
    p = rng.uniform(0.05, 1.0, nv).astype(np.float32)
    p[::7] = 1.0
    p[3::11] = np.float32(2.0 ** -33)     # a threshold of 0: never drawn
    log(f"design draws {name} R={R}")
    got = pair.design_inclusion(_t(off), _t(p), 2 ** 63 + 5, 9, R, gmax, nv=nv)
    torch.cuda.synchronize()
    want = oracle.design_inclusion(off, p, 2 ** 63 + 5, 9, R, gmax)
    assert int(got["status"].item()) == 0
    for key in ("mask", "pi", "edge_count", "completed"):
        assert np.array_equal(got[key].cpu().numpy(), want[key]), key


@pytest.mark.parametrize("name,R", [("edges", 1), ("full", 256), ("full", 257), ("one", 4096),
                                    ("one", 4097), ("twos", 125)])
def test_design_draws_without_a_rho_block(name, R):
    """Wide groups without a rho block, as many (replicate, prompt) pairs as a wave
    each still takes (4096), and more."""
    off = _offsets(name)
    nv, gmax = int(off[-1]), max(SIZES[name])
    p = np.random.default_rng(R).uniform(0.05, 1.0, nv).astype(np.float32)
    log(f"design draws without rho {name} R={R}")
    got = pair.design_inclusion(_t(off), _t(p), 12, 3, R, gmax, nv=nv, want_pi=False)
    torch.cuda.synchronize()
    want = oracle.design_inclusion(off, p, 12, 3, R, gmax)
    assert int(got["status"].item()) == 0
    for key in ("mask", "edge_count", "completed"):
        assert np.array_equal(got[key].cpu().numpy(), want[key]), key


@pytest.mark.parametrize("R", [1, 40])
def test_design_optional_outputs_and_bad_prompts(R):
    """Each output alone is what it is beside the others; a malformed prompt and
    probabilities outside (0, 1] leave the other prompts' draws as they are,
    and a malformed prompt's mask and counts untouched."""
    off = np.array([0, 5, 6, 14, 90, 110], dtype=np.int64)     # groups of 1 and 76 are malformed
    nv, gmax, B = 110, 20, 5
    p = np.random.default_rng(1).uniform(0.3, 1.0, nv).astype(np.float32)
    p[2], p[8], p[95] = 0.0, np.nan, 1.5

    def call(names):
        out = {"mask": torch.full((R, nv), 7, dtype=torch.uint8, device=DEV),
               "pi": torch.full((B, gmax, gmax), 7.0, device=DEV),
               "edge_count": torch.full((R, B), 7, dtype=torch.int32, device=DEV),
               "completed": torch.full((R, B), 7, dtype=torch.int32, device=DEV)}
        out = {k: v for k, v in out.items() if k in names}
        st = torch.zeros(1, dtype=torch.int32, device=DEV)
        pair.pair_design_inclusion(B, nv, gmax, _t(off), _t(p), 3, 0, R, d_status=st, **out)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}, int(st.item())

    every, st = call(("mask", "pi", "edge_count", "completed"))
    assert st == pair.ST_P_RANGE | pair.ST_BAD_GROUP
    for key in every:
        alone, st1 = call((key,))
        assert np.array_equal(alone[key], every[key], equal_nan=True), key
        assert st1 & pair.ST_BAD_GROUP
    m = every["mask"]
    for b in (1, 3):
        assert np.all(m[:, off[b]:off[b + 1]] == 7) and np.all(every["pi"][b] == 0.0)
        assert np.all(every["completed"][:, b] == 7) and np.all(every["edge_count"][:, b] == 7)
    for b in (0, 2, 4):
        k = m[:, off[b]:off[b + 1]].sum(axis=1)
        assert np.array_equal(every["completed"][:, b], k)
        assert np.array_equal(every["edge_count"][:, b], k * (k - 1) // 2)
    assert np.all(m[:, [2, 8, 95]] == 0)
    ok = (p > 0) & (p <= 1)
    rows = np.r_[0:5, 6:14, 90:110]     # prompts 0, 2 and 4
    q = np.where(ok, p, np.float32(0.5)).astype(np.float32)[rows]
    want = oracle.design_inclusion(np.array([0, 5, 13, 33]), q, 3, 0, R, gmax, prompt_id=[0, 2, 4])
    assert np.array_equal(m[:, rows][:, ok[rows]], want["mask"][:, ok[rows]])


@pytest.mark.parametrize("name", ["edges", "one", "twos"])
@pytest.mark.parametrize("R", [1, 63, 64, 65, 256, 257])
def test_fixed_size_draws(name, R):
    off = _offsets(name)
    nv, gmax, B = int(off[-1]), max(SIZES[name]), len(SIZES[name])
    rng = np.random.default_rng(R)
    odds = np.exp(rng.normal(0.0, 1.5, nv))
    n = np.array([rng.integers(0, g + 1) for g in SIZES[name]], dtype=np.int32)
    n[-1] = SIZES[name][-1] - 1
    log(f"fixed-size draws {name} R={R}")
    got = pair.cps_draw(_t(off), _t(odds), _t(n), 2 ** 62 + 1, 4, R, gmax, nv=nv)
    torch.cuda.synchronize()
    assert int(got["status"].item()) == 0
    assert np.array_equal(got["mask"].cpu().numpy(), oracle.cps_draw(off, odds, n, 2 ** 62 + 1, 4, R))
    assert np.array_equal(got["edge_count"].cpu().numpy(), np.tile(n * (n - 1) // 2, (R, 1)))
