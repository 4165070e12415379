"""The HIP kernels at the edges of their tiles: batches of lines and slabs of
planes of the rate kernel, ragged tiles of the Re transform, counts around a
tile of the surrogate's inference and around a block of the moments, calls
that only count.

Tolerances.  Two runs that differ in how a state's terms are grouped form the
same terms and add them in FP64 in another order: at most some 1e5 positive
terms, so 1e-12.  Against the oracle 1e-10 in FP64 and 1e-4 in FP32, as for
the other grids; moments 1e-12 of the largest element, as a reduction of the
same data; inference 1e-4 of the largest value (FP32 dot products of 128).
"""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import log, params_for, gpu_run, compare_rates, rel_err
from synth import make_system, workload
from oracle import Oracle
from oracle import mlp as ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# lines per batch 15, 16, 9 + 8, 11 + 10; with every state in the window the
# slabs hold all planes, with a few k points one plane each
@pytest.mark.parametrize("name,N,prec,temps", [
    ("toy_sc_8", 15, "fp64", [300.0]), ("toy_sc_8", 16, "fp64", [200.0, 300.0, 400.0]),
    ("toy_sc_8", 17, "fp64", [300.0, 500.0]), ("toy_sc_8", 17, "fp32", [300.0]),
    ("toy_sc_8", 21, "fp32", [200.0, 300.0, 400.0, 500.0]), ("al_fcc_100", 19, "fp32", [300.0, 500.0]),
    ("al_fcc_100", 20, "bf16x3", [300.0]), ("al_fcc_100", 18, "fp64", [300.0])])
def test_slabs_and_batches(torch_cuda, name, N, prec, temps):
    from paper_2306_16493_amd import Context
    w = workload(name, N)
    s = make_system(w.system)
    ctx = Context(s)
    full = gpu_run(ctx, params_for(ctx, w, s, N, precision=prec, temps=temps)[0])
    ks = np.unique(full["state_k"])
    ks = np.unique(np.concatenate([ks[:1], ks[-1:], np.random.default_rng(N).choice(ks, 3, replace=False)]))
    p, (N, mu, lo, hi) = params_for(ctx, w, s, N, precision=prec, temps=temps, k_subset=ks)
    few = gpu_run(ctx, p)
    sel = np.isin(full["state_k"], ks)
    assert np.array_equal(full["state_k"][sel], few["state_k"]) and np.array_equal(full["state_n"][sel], few["state_n"])
    assert np.array_equal(full["energy"][sel], few["energy"]) and np.array_equal(full["vel"][sel], few["vel"])
    err = np.max(np.abs(full["inv_tau"][:, sel] - few["inv_tau"]) / np.maximum(few["inv_tau"], 1e-300))
    log(f"[slabs] {name} {N} {prec}: {few['counts']['n_states']} of {full['counts']['n_states']} states, err {err:.1e}")
    assert err < 1e-12
    r = Oracle(s).run(N, mu, temps, w.eta, lo, hi, w.band_lo, w.band_hi, k_subset=ks)
    compare_rates(few, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"], tol=1e-10 if prec == "fp64" else 1e-4)
    assert few["counts"]["n_kq"] == r["n_kq"] and few["counts"]["n_terms"] == int(r["n_terms"].sum())
    ctx.close()


@pytest.mark.parametrize("name,N", [("mini_w1", 2), ("mini_w2a2", 1), ("mini_w8", 2), ("toy_sc", 2)])
def test_smallest_grids(torch_cuda, name, N):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    mu, temps = s.mu_centroid, [300.0]
    ctx = Context(s)
    g = gpu_run(ctx, ctx.params(N, mu, temps, 0.5, -1e3, 1e3))
    r = Oracle(s).run(N, mu, temps, 0.5, -1e3, 1e3)
    compare_rates(g, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"])
    assert g["counts"]["n_terms"] == int(r["n_terms"].sum())
    ctx.close()


# K = n_re * n_wann not a multiple of the tile's 16, numbers of states around
# the tile's 64
@pytest.mark.parametrize("name,n_re,n_k,prec", [
    ("mini_w1", 61, 1, "fp64"), ("mini_w1", 61, 65, "fp32"), ("mini_w2a2", 59, 32, "fp64"),
    ("mini_w2a2", 59, 33, "fp32"), ("mini_w8", 63, 8, "fp64"), ("mini_w4a2", 3, 17, "fp64")])
def test_transform_tiles(torch_cuda, name, n_re, n_k, prec):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    s = dataclasses.replace(s, re=np.ascontiguousarray(s.re[:n_re]), gw=np.ascontiguousarray(s.gw[:n_re]))
    N, mu, temps = 5, s.mu_centroid, [300.0]
    ks = np.random.default_rng(n_k).choice(N ** 3, n_k, replace=False)
    ctx = Context(s)
    g = gpu_run(ctx, ctx.params(N, mu, temps, 0.05, -1e3, 1e3, precision=prec, k_subset=ks))
    r = Oracle(s).run(N, mu, temps, 0.05, -1e3, 1e3, k_subset=np.sort(ks))
    assert g["counts"]["n_states"] == n_k * s.nw
    compare_rates(g, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"], tol=1e-10 if prec == "fp64" else 1e-4)
    ctx.close()


def test_counting_calls(torch_cuda):
    """A call without room for a state counts as the full call does, and an
    empty window still counts the excluded modes."""
    from paper_2306_16493_amd import Context
    w = workload("al_fcc_100", 9)
    s = make_system(w.system)
    ctx = Context(s)
    p, (N, mu, lo, hi) = params_for(ctx, w, s, 9)
    n = ctx.count_states(p)  # the tables of a count hold energies alone: the next call builds its own
    res, _ = ctx.scattering_rates(p, capacity=n)
    assert res.counts["n_states"] == n > 0
    again, _ = ctx.scattering_rates(p, capacity=n + 7)
    assert np.array_equal(res.inv_tau.cpu().numpy(), again.inv_tau.cpu().numpy())
    empty, _ = ctx.scattering_rates(params_for(ctx, w, s, 9, window=(500.0, 600.0))[0], capacity=0)
    assert empty.counts["n_states"] == 0
    assert empty.counts["n_excluded_modes"] == res.counts["n_excluded_modes"] > 0
    ctx.close()


@pytest.mark.parametrize("n,nt", [(1, 1), (255, 2), (257, 3), (4096, 4), (65537, 3)])
def test_moments_any_count(torch_cuda, n, nt):
    from paper_2306_16493_amd import Context
    torch = torch_cuda
    s = make_system("toy_sc")
    ctx = Context(s)
    rng = np.random.default_rng(n)
    e, v = rng.normal(0, 0.2, n), rng.normal(0, 1e6, (n, 3))
    it = 10.0 ** rng.uniform(11, 15, (nt, n))
    it[:, n // 2 + 1::7] = 0.0  # states without a rate are left out
    temps = [100.0, 300.0, 500.0, 700.0][:nt]
    dev = [torch.tensor(x, device="cuda") for x in (e, v, it.reshape(-1))]
    got = ctx.transport(*dev, 0.01, temps, 1000)
    sig = ctx.conductivity(*dev, 0.01, temps, 1000)
    want = Oracle(s).transport(e, v, it, 0.01, temps, 1000)
    assert np.array_equal(sig, got[0])
    if n >= 3:  # the Seebeck coefficient inverts sigma
        for a, b in zip(got, want):
            assert rel_err(a, b) < 1e-12
    else:
        assert rel_err(got[0], want[0]) < 1e-12
    ctx.close()


# below, at and above a tile of 64; more tiles than workgroups walk at a time
@pytest.mark.parametrize("n,nout,members", [(1, 1, 1), (63, 2, 2), (64, 4, 1), (65, 3, 5), (1300, 1, 64), (7000, 1, 5)])
def test_predict_any_count(torch_cuda, n, nout, members):
    from paper_2306_16493_amd import Context
    from paper_2306_16493_amd.eph import Mlp
    torch = torch_cuda
    ctx = Context(make_system("toy_sc"))
    m = Mlp(ctx, members=members, n_out=nout, seed=11)
    rng = np.random.default_rng(n)
    x = rng.normal(0.3, 2.0, (7000, ref.NIN)).astype(np.float32)
    y = rng.normal(1.0, 3.0, (7000, nout)).astype(np.float32)
    xt, yt = torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")
    m.train(xt, yt, steps=1, batch=32, lr=1e-3)  # sets the normalisation
    pr = m.get_params()
    xm, xs, ym, ys = (f(a.astype(np.float64), axis=0) for a in (x, y) for f in (np.mean, np.std))
    got = m.predict(xt[:n]).cpu().numpy()
    assert got.shape == (members, n, nout)
    for e in {0, members - 1}:
        want = ref.forward(pr[e].astype(np.float64), (x[:n] - xm) / xs, nout)[0] * ys + ym
        assert np.max(np.abs(got[e] - want)) < 1e-4 * np.max(np.abs(want)) + 1e-5
    m.close()
    ctx.close()
