"""The direct Bloch sum (R lists that fill no box) for every number of bands
and modes, with lists around the length of its runs of phases (32 vectors for 3
and 4 columns, 64 for 6 and 8), against the oracle; and counts against lists for
both forms of the sum: a count solves for the energies alone, in a kernel of its
own, and must see them to the last bit.

Tolerances as for the other grids: energies, velocities away from degeneracies
and rates 1e-10.
"""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import log, gpu_run, compare_rates, degenerate_mask, rel_err
from synth import make_system
from synth.systems import _draw_ham, _draw_ifc, _sc
from oracle import Oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def sparse_vectors(rng, npairs):
    """R = 0, +-(7, 0, 0) and npairs - 1 more pairs: too long along R1 for a box."""
    seen = {(7, 0, 0)}
    while len(seen) < npairs:
        v = tuple(int(x) for x in rng.integers(-4, 5, 3))
        if v > (0, 0, 0):
            seen.add(v)
    pairs = [list(v) for v in sorted(seen)]
    return np.array([[0, 0, 0]] + pairs + [[-x for x in v] for v in pairs], np.int32)


def sparse(name, nw, npairs):
    """A small model whose H and D lists take the direct sum."""
    s = make_system(name)
    rng = np.random.default_rng([nw, npairs])
    r = sparse_vectors(rng, npairs)
    w = np.ones(len(r))
    ham = _draw_ham(rng, _sc(1.0), r, nw)  # decay over 1 A per cell: the far vectors stay visible
    ifc = _draw_ifc(rng, _sc(1.0), s.tau * 0.3, s.mass, r, w, 0.040)
    return dataclasses.replace(s, nw=nw, rh=r, rh_w=w, ham=ham, rd=r, rd_w=w, ifc=ifc,
                               gw=np.ascontiguousarray(s.gw[..., :nw, :nw]),
                               mu_centroid=float(np.real(np.trace(ham[0]))) / nw)


@pytest.mark.parametrize("name,nw,npairs,N", [
    ("mini_w1", 1, 7, 6), ("mini_w2a2", 2, 33, 5), ("toy_sc", 4, 15, 6), ("toy_sc", 4, 16, 5), ("mini_w4a2", 4, 31, 4),
    ("mini_w8", 8, 31, 4), ("mini_w8", 8, 32, 5), ("mini_w4a2", 4, 70, 5)])
def test_direct_sum_vs_oracle(torch_cuda, name, nw, npairs, N):
    from paper_2306_16493_amd import Context
    s = sparse(name, nw, npairs)
    mu, temps, eta = s.mu_centroid, [300.0], 0.05
    ctx = Context(s)
    g = gpu_run(ctx, ctx.params(N, mu, temps, eta, -1e3, 1e3))
    r = Oracle(s).run(N, mu, temps, eta, -1e3, 1e3)
    log(f"[direct] {nw} bands, {s.nmodes} modes, {len(s.rh)} vectors, {N}^3: energy err {rel_err(g['energy'], r['energy']):.1e}")
    assert np.array_equal(g["state_k"], r["state_k"]) and np.array_equal(g["state_n"], r["state_n"])
    assert rel_err(g["energy"], r["energy"]) < 1e-10
    nd = ~degenerate_mask(r["tables"][0], r["state_k"], r["state_n"])
    assert np.max(np.abs(g["vel"][nd] - r["vel"][nd])) <= 1e-10 * np.abs(r["vel"]).max()
    compare_rates(g, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"])
    assert g["counts"]["n_terms"] == int(r["n_terms"].sum())
    ctx.close()


@pytest.mark.parametrize("name,nw,npairs,N", [
    ("mini_w1", 1, 0, 9), ("mini_w2a2", 2, 0, 8), ("toy_sc", 4, 0, 9), ("al_fcc", 4, 0, 10), ("si_fcc", 8, 0, 7),
    ("mini_w1", 1, 20, 9), ("mini_w2a2", 2, 20, 8), ("toy_sc", 4, 20, 9), ("mini_w8", 8, 40, 6)])
def test_counts_see_the_listed_energies(torch_cuda, name, nw, npairs, N):
    """Windows that end at a state's energy, from either side."""
    from paper_2306_16493_amd import Context
    s = sparse(name, nw, npairs) if npairs else make_system(name)
    ctx = Context(s)
    par = lambda lo, hi: ctx.params(N, 0.0, [300.0], 0.02, lo, hi)
    e = ctx.select_states(par(-1e3, 1e3))[2].cpu().numpy()
    for x in np.random.default_rng(N).choice(e, 100, replace=False):
        assert ctx.count_states(par(x, 1e3)) == np.sum(e >= x)
        assert ctx.count_states(par(-1e3, x)) == np.sum(e <= x)
    ctx.close()
