"""Gradients of rows that end inside a piece of four columns, at the edges of
tiles and of the narrowest rows: padded and unpadded, aligned or not.  The
row's padding holds NaN.

Bound: n fp32 multiply-adds per column in some order, each rounding once and
within 2^-24 of the sum of magnitudes, and the division by B: (n + 1) 2^-24."""
import numpy as np
import pytest
import torch

import paper_2608_11368_amd as pair
from tests.gpu_util import DEV, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 7, 1023, 1025, 2047, 2049, 2050, 4095, 4097, 4099,
                               8191, 12291])
@pytest.mark.parametrize("pad", [0, 13])
def test_ragged_width(D, dtype, pad):
    unit = 16 // (4 if dtype == torch.float32 else 2)
    ld = (D + unit - 1) // unit * unit + (unit if pad else 0)
    sizes = [2, 64, 13, 9, 30]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    nv = int(off[-1])
    gen = torch.Generator().manual_seed(D)
    full = torch.full((nv, ld), float("nan"), dtype=dtype)
    full[:, :D] = torch.randn(nv, D, generator=gen).to(dtype)
    c = torch.randn(nv, generator=gen)
    c[torch.rand(nv, generator=gen) < 0.4] = 0.0
    c[off[3]:off[4]] = 0.0                          # a prompt without coefficients
    live = (c != 0).numpy()
    full[torch.from_numpy(~live)] = float("nan")    # rows without a coefficient are not read
    log(f"ragged width D={D} ld={ld} {dtype}")
    s = full.to(DEV)[:, :D]
    o, cd = torch.from_numpy(off).to(DEV), c.to(DEV)
    per = pair.weighted_grad(o, s, cd, nv=nv)["out"].cpu().double()
    mean = pair.weighted_grad(o, s, cd, nv=nv, reduce=True)["out"].cpu().double()
    x = torch.nan_to_num(full[:, :D].double())
    terms = c.double()[:, None] * x
    for b in range(len(sizes)):
        t = terms[off[b]:off[b + 1]]
        assert torch.all((per[b] - t.sum(0)).abs() <= (sizes[b] + 1) * 2.0 ** -24 * t.abs().sum(0)), b
    bound = (nv + 1) * 2.0 ** -24 * terms.abs().sum(0) / len(sizes)
    assert torch.all((mean - terms.sum(0) / len(sizes)).abs() <= bound)
