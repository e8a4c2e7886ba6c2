"""CPU check of the rounding bounds that the random audit tests hold every e_r
and bias norm to.  The audit's arithmetic, an fp32 fold (weights, sums over the
partners in order, centring) and K = S S^T from fp32 sums of 128 columns added
in fp64, is emulated in numpy on the oracle's own draws; its errors must stay
within the bounds, single-column cases whose terms cancel among them.  And the
bounds must be near enough to see a lost digit: the same arithmetic with its
normaliser, its mean or K off by 2^-14 exceeds them."""
import numpy as np
import pytest

import oracle
from tests import test_gpu_random as T

RUN = 128


def _audit(c, R, off_norm=1.0, off_mean=1.0, off_gram=1.0):
    """(e_r [B][R], bias [B]) of the emulation and the exact ones."""
    off = c["offsets"]
    od = oracle.design_inclusion(off, c["p"], c["seed"], c["rep0"], R, c["gmax"])
    a, _ = oracle.pair_coeffs(off, c["rewards"])
    S = (c["host"].astype(np.uint32) << 16).view(np.float32)
    B = off.size - 1
    e, bias, want_e, want_b = np.zeros((B, R)), np.zeros(B), np.zeros((B, R)), np.zeros(B)
    for b in range(B):
        o0, o1 = int(off[b]), int(off[b + 1])
        g, sb = o1 - o0, S[o0:o1]
        r, p = c["rewards"][o0:o1], c["p"][o0:o1]
        K = np.zeros((g, g))
        for k in range(0, sb.shape[1], RUN):
            run = np.zeros((g, g), dtype=np.float32)
            for x in sb[:, k:k + RUN].T:
                run += x[:, None] * x[None, :]
            K += run
        K *= off_gram
        W = (r[:, None] - r[None, :]) / (p[:, None] * p[None, :])
        np.fill_diagonal(W, 0.0)
        x = np.zeros((R, g))
        for q in range(R):
            J = od["mask"][q, o0:o1].astype(np.float32)
            k = int(J.sum())
            fold = np.zeros(g, dtype=np.float32)
            if k >= 2:
                for j in range(g):
                    fold += J[j] * W[:, j]
                fold *= J
                mean = np.float32(np.sum(fold, dtype=np.float32) / np.float32(k)) * np.float32(off_mean)
                mean += np.float32(off_mean - 1.0) * np.abs(fold).max()
                fold = (fold - mean) * J
            x[q] = fold.astype(np.float64) * (off_norm / (g * (g - 1)))
        t = a[o0:o1].astype(np.float32).astype(np.float64)
        d = x - t
        e[b] = np.maximum(np.einsum("ri,ij,rj->r", d, K, d), 0.0).astype(np.float32)
        dbar, s64 = d.mean(axis=0), sb.astype(np.float64)
        form = dbar @ K @ dbar
        if 64.0 * form >= (dbar ** 2 * np.diag(K)).sum():
            bias[b] = np.sqrt(form)
        else:
            bias[b] = np.linalg.norm(dbar @ s64)
        exact = np.stack([oracle.pair_coeffs(off, c["rewards"], od["mask"][q], od["pi"])[0][o0:o1]
                          for q in range(R)]) - a[o0:o1]
        want_e[b] = np.sum((exact @ s64) ** 2, axis=1)
        want_b[b] = np.linalg.norm(exact.mean(axis=0) @ s64)
    return e, bias, want_e, want_b


def _shares(monkeypatch, case_id, **off):
    monkeypatch.setattr(T, "DEV", "cpu")
    rng = np.random.default_rng(9100 + case_id)
    c = T._case(rng, 5, (1, 33, 500, 2047), bf16=True)
    R = int(rng.choice([1, 31, 33, 64]))
    e, bias, want_e, want_b = _audit(c, R, **off)
    e_bound, b_bound = T._audit_rounding_bounds(c, R)
    floor = 1e-300
    dead = want_e.max(axis=1) == 0.0     # equal rewards: zero error, zero bound
    if not off:
        assert np.all(e[dead] == 0.0) and np.all(e_bound[dead] == 0.0)
    return (np.max(np.abs(e - want_e) / np.maximum(e_bound, floor)),
            np.max(np.abs(bias - want_b) / np.maximum(b_bound, floor)))


@pytest.mark.parametrize("case_id", [5, 1062, 1064, 1171, 1192] + list(range(2000, 2012)))
def test_emulated_errors_are_within_the_bounds(monkeypatch, case_id):
    e, bias = _shares(monkeypatch, case_id)
    print(f"largest error / bound: e_r {e:.3f}, bias {bias:.3f}")
    assert e <= 1.0 and bias <= 1.0


@pytest.mark.parametrize("what", ["off_norm", "off_mean", "off_gram"])
def test_lost_digits_exceed_the_bounds(monkeypatch, what):
    shares = [_shares(monkeypatch, k, **{what: 1.0 + 2.0 ** -14}) for k in range(2000, 2006)]
    print([f"{e:.1f} {b:.1f}" for e, b in shares])
    assert max(max(x) for x in shares) > 2.0
