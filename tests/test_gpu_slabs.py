"""The rate kernel's slabs of q3 planes: slabs of one and of several planes, and
launches that take all slabs, some (the last one fewer) or one at a time.

A state's sums are added slab by slab in order, however many a launch takes:
results, counts and transition rates are the same to the last bit.  Slabs of
several planes group the terms otherwise: 1e-12, as some 1e5 positive terms in
FP64.
"""
import re

import numpy as np
import pytest

from gpu_helpers import log, gpu_run, compare_rates
from synth import make_system
from oracle import Oracle

pytestmark = pytest.mark.gpu

ROOM = 8 << 30  # a budget that holds everything: with one, a launch's sums keep to the plan's share


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def slab_rule(N, ns, fp64):
    """(planes per slab, slabs) by the library's rule."""
    planes = max(1, min(((10000 if fp64 else 20000) + N * N // 2) // (N * N), ns * N // 8192, N))
    return planes, -(-N // planes)


def pick(N, n, seed):
    return np.sort(np.random.default_rng(seed).choice(N ** 3, n, replace=False))


def launches(ctx, call):
    ctx.set_profiling(True)
    out = call()
    return out, ctx.stage_times()


def least_budget(call):
    """(fixed bytes, bytes per state, least budget) from what a refusal says."""
    from paper_2306_16493_amd import EphError
    said = "(0 bytes)"
    for _ in range(2):
        try:
            call(int(re.search(r"\((\d+) bytes\)", said).group(1)) + 1)
        except EphError as e:
            said = str(e)
    m = re.search(r"minimum of (\d+) bytes \((\d+) bytes of tables and lists plus (\d+) bytes per state", said)
    assert m, said
    return int(m.group(2)), int(m.group(3)), int(m.group(1))


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# k points, temperatures: one plane per slab and a prime number of slabs, two
# planes per slab with one left over
@pytest.mark.parametrize("name,N,n_k,temps,prec", [
    ("toy_sc", 17, 75, [300.0], "fp64"), ("toy_sc", 29, 150, [300.0, 500.0], "fp64"),
    ("toy_sc", 29, 150, [300.0], "fp32"), ("mini_w8", 17, 36, [200.0, 300.0, 400.0], "fp64"),
    ("mini_w4a2", 17, 75, [300.0], "fp32"), ("mini_w2a2", 31, 200, [300.0], "bf16x3")])
def test_launches_of_some_slabs(torch_cuda, name, N, n_k, temps, prec):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    ctx = Context(s)
    ks = pick(N, n_k, N)
    par = lambda budget: ctx.params(N, s.mu_centroid, temps, 0.05, -1e3, 1e3, precision=prec, k_subset=ks,
                                    mem_budget_bytes=budget)
    planes, slabs = slab_rule(N, n_k * s.nw, prec == "fp64")
    one, t1 = launches(ctx, lambda: gpu_run(ctx, par(0)))
    some, t2 = launches(ctx, lambda: gpu_run(ctx, par(ROOM)))
    log(f"[slabs] {name} {N}^3 {prec}: {n_k * s.nw} states, {slabs} slabs of {planes}, {t1['rates_launches']} and "
        f"{t2['rates_launches']} launches")
    assert t1["rates_launches"] == 1 and 1 < t2["rates_launches"] < slabs
    per = [p for p in range(2, slabs) if -(-slabs // p) == t2["rates_launches"]]
    assert per and all(slabs % p for p in per)  # the last launch takes fewer
    same((one["inv_tau"], one["energy"]), (some["inv_tau"], some["energy"]))
    assert one["counts"] == some["counts"]
    # and in batches of states
    fixed, per_state, _ = least_budget(lambda b: gpu_run(ctx, par(b)))
    batched, t3 = launches(ctx, lambda: gpu_run(ctx, par(fixed + per_state * (n_k * s.nw // 3))))
    assert t3["xform_launches"] >= 3 and t3["rates_launches"] == t3["xform_launches"] * t2["rates_launches"]
    same((one["inv_tau"],), (batched["inv_tau"],))
    assert one["counts"] == batched["counts"]
    ctx.close()


# as above for transition rates: all slabs in one launch (counted once), some
# (counted again per launch), in batches through the staging buffer
@pytest.mark.parametrize("name,N,n_k,temps", [("toy_sc", 17, 60, [300.0]), ("toy_sc", 29, 150, [300.0, 500.0]),
                                              ("mini_w4a2", 17, 60, [300.0]), ("mini_w8", 17, 30, [300.0])])
def test_transition_rates_by_launches(torch_cuda, name, N, n_k, temps):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    ctx = Context(s)
    ks = pick(N, n_k, N + 1)
    par = lambda budget: ctx.params(N, s.mu_centroid, temps, 0.05, -1e3, 1e3, k_subset=ks, mem_budget_bytes=budget)
    planes, slabs = slab_rule(N, n_k * s.nw, True)
    (res, gam), t1 = launches(ctx, lambda: ctx.rates_gamma(par(0)))
    (res2, gam2), t2 = launches(ctx, lambda: ctx.rates_gamma(par(ROOM)))
    info = gam.info()
    log(f"[slabs] {name} {N}^3: {n_k * s.nw} states, {info['nnz']} rates, {slabs} slabs of {planes}, "
        f"{t1['rates_launches']} and {t2['rates_launches']} launches")
    assert t1["rates_launches"] == 1 and 1 < t2["rates_launches"] < slabs
    assert ctx.gamma_estimate(par(0))[1] == ctx.gamma_estimate(par(ROOM))[1] == info["nnz"]
    rows, it = gam.rows(), res.inv_tau.cpu().numpy()
    same(rows, gam2.rows())
    same((it,), (res2.inv_tau.cpu().numpy(),))
    assert res.counts == res2.counts
    least = least_budget(lambda b: ctx.rates_gamma(par(b)))[2]
    (res3, gam3), t3 = launches(ctx, lambda: ctx.rates_gamma(par(least + 2 * (4 + 8 * len(temps)) * (info["nnz"] // 3))))
    assert gam3.info()["on_host"] and t3["xform_launches"] > 1
    same(rows, gam3.rows())
    same((it,), (res3.inv_tau.cpu().numpy(),))
    # rates between the same states from slabs of one plane
    few = ks[::3]
    assert slab_rule(N, len(few) * s.nw, True)[0] == 1
    res4, gam4 = ctx.rates_gamma(ctx.params(N, s.mu_centroid, temps, 0.05, -1e3, 1e3, k_subset=few))
    keep = np.isin(res.state_k.cpu().numpy(), few)
    compare_subset(rows, gam4.rows(), keep)
    for g in (gam, gam2, gam3, gam4):
        g.close()
    ctx.close()


def compare_subset(rows, sub, keep):
    """Rows of the kept states among the kept states, against sub's."""
    rs, col, val = rows
    rs4, col4, val4 = sub
    new = np.cumsum(keep) - 1
    for j, i in enumerate(np.flatnonzero(keep)):
        c, v = col[rs[i]:rs[i + 1]], val[:, rs[i]:rs[i + 1]]
        v, c = v[:, keep[c]], new[c[keep[c]]]
        o, o4 = np.argsort(c), np.argsort(col4[rs4[j]:rs4[j + 1]])
        assert np.array_equal(c[o], col4[rs4[j]:rs4[j + 1]][o4])
        if len(c):
            w = val4[:, rs4[j]:rs4[j + 1]][:, o4]
            assert np.max(np.abs(v[:, o] - w)) <= 1e-12 * np.abs(w).max()


# several planes per slab (all of them on these grids) in every shape, FP64 with
# 48 channels and FP32 with 12 reading X once for two of them
@pytest.mark.parametrize("name,N,prec", [
    ("si_fcc", 12, "fp64"), ("si_fcc", 11, "fp32"), ("mini_w8", 13, "fp64"), ("mini_w8", 13, "fp32"),
    ("mini_w4a2", 13, "fp64"), ("mini_w4a2", 13, "bf16x3"), ("mini_w2a2", 16, "fp64"), ("mini_w2a2", 15, "fp32"),
    ("mini_w1", 19, "fp64"), ("mini_w1", 19, "fp32"), ("toy_sc", 17, "fp32")])
def test_slabs_of_several_planes(torch_cuda, name, N, prec):
    from paper_2306_16493_amd import Context
    s = make_system(name)
    ctx = Context(s)
    mu, temps, eta = s.mu_centroid, [300.0, 500.0], 0.05
    full = gpu_run(ctx, ctx.params(N, mu, temps, eta, -1e3, 1e3, precision=prec))
    ks = pick(N, 3, N)
    few = gpu_run(ctx, ctx.params(N, mu, temps, eta, -1e3, 1e3, precision=prec, k_subset=ks))
    assert slab_rule(N, full["counts"]["n_states"], prec == "fp64")[0] > 1
    assert slab_rule(N, few["counts"]["n_states"], prec == "fp64")[0] == 1
    sel = np.isin(full["state_k"], ks)
    err = np.max(np.abs(full["inv_tau"][:, sel] - few["inv_tau"]) / np.maximum(few["inv_tau"], 1e-300))
    log(f"[slabs] {name} {N}^3 {prec}: {full['counts']['n_states']} states, several planes and one differ by {err:.1e}")
    assert err < 1e-12
    r = Oracle(s).run(N, mu, temps, eta, -1e3, 1e3, k_subset=ks[:1])
    at = np.isin(few["state_k"], ks[:1])
    first = dict(inv_tau=few["inv_tau"][:, at])
    compare_rates(first, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"], tol=1e-10 if prec == "fp64" else 1e-4)
    ctx.close()


def test_transition_rates_over_the_planes_of_a_slab(torch_cuda):
    """48 channels: two planes per slab, the second from LDS, positions running
    on over the planes."""
    from paper_2306_16493_amd import Context
    s = make_system("si_fcc")
    N = 12
    ks = pick(N, 172, 5)
    few = ks[::3]
    assert slab_rule(N, len(ks) * s.nw, True)[0] == 2 and slab_rule(N, len(few) * s.nw, True)[0] == 1
    ctx = Context(s)
    par = lambda k: ctx.params(N, s.mu_centroid, [300.0], 0.01, -1e3, 1e3, k_subset=k)
    res, gam = ctx.rates_gamma(par(ks))
    res4, gam4 = ctx.rates_gamma(par(few))
    keep = np.isin(res.state_k.cpu().numpy(), few)
    compare_subset(gam.rows(), gam4.rows(), keep)
    a, b = res.inv_tau.cpu().numpy()[:, keep], res4.inv_tau.cpu().numpy()
    assert np.max(np.abs(a - b) / b) < 1e-12
    gam.close()
    gam4.close()
    ctx.close()
