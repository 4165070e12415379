"""Occupation weights where emission is blocked: states at the top of filled
bands (f = 1 to the last bit) at 2 K, where a transition rate is what the tail
of the absorption Gaussian leaves.

Tolerance.  A tail e^{-(x/eta)^2}, x up to 6 eta, of energies good to 1e-14 eV
has a relative error of 12 x 1e-14 / 0.02 = 6e-12, |g|^2 one of some 1e-11:
1e-9.  Below 1e-17 of the row at 300 K an entry is not compared: the Bose
factor of the softest mode there, e^{-7.3 meV / k_B 2 K} = 4e-19, is lost in
the oracle's 1 + N - f and kept here.
"""
import numpy as np
import pytest

from gpu_helpers import log
from synth import make_system
from oracle import Oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("name,N", [("toy_sc", 8), ("mini_w4a2", 5), ("mini_w8", 5)])
def test_blocked_emission_leaves_the_absorption_tail(torch_cuda, name, N):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    o = Oracle(s)
    eps, evec, _ = o.electrons(N)
    om, u, _ = o.phonons(N)
    top, eta, temps = eps.max(), 0.02, [2.0, 300.0]
    mu, lo, hi = top + 1.0, top - 0.4, top + 1e-7
    sk, sn = o.select_states(eps, 0, -1, lo, hi)
    ref = o.gamma(N, eps, evec, om, u, sk, sn, mu, temps, eta)
    ctx = Context(s)
    res, gam = ctx.rates_gamma(ctx.params(N, mu, temps, eta, lo, hi))
    rs, col, val = gam.rows()
    assert np.array_equal(res.state_k.cpu().numpy(), sk) and np.array_equal(res.state_n.cpu().numpy(), sn)
    index = -np.ones(N ** 3 * s.nw, np.int64)
    index[sk.astype(np.int64) * s.nw + sn] = np.arange(len(sk))
    worst, tails = 0.0, 0
    for i in range(len(sk)):
        c = index[ref["fin"][ref["row_start"][i]:ref["row_start"][i + 1]]]
        want = ref["val"][ref["row_start"][i]:ref["row_start"][i + 1]][c >= 0]
        order, got_order = np.argsort(c[c >= 0]), np.argsort(col[rs[i]:rs[i + 1]])
        assert np.array_equal(c[c >= 0][order], col[rs[i]:rs[i + 1]][got_order])
        if not len(want):
            continue
        floor = 1e-17 * want[:, 1].max()
        want, got = want[order, 0], val[0, rs[i]:rs[i + 1]][got_order]
        worst = max(worst, float(np.max(np.abs(got - want) / np.maximum(want, floor))))
        tails += int(np.sum((want > floor) & (want < 1e6 * floor)))
    log(f"[occupations] {name} {N}^3: {len(sk)} states, {len(col)} rates, {tails} tails, max rel err {worst:.1e}")
    assert tails > 10
    assert val.min() >= 0.0
    assert worst < 1e-9
    gam.close()
    ctx.close()
