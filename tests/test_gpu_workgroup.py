"""The workgroup form of the rate kernel, which serves every Rp box but the
cubes of edge 4 and 6, at each (orbitals, modes) shape: models cut to a 3^3 or
3 x 4 x 4 box, or to one orbital, against the oracle.

Tolerances as for the other grids: 1e-10 per state in FP64, 1e-4 in FP32 and BF16x3,
counts equal.
"""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import log, gpu_run, compare_rates
from synth import make_system
from oracle import Oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def cut(s, box, nw=None):
    """The model with its Rp set cut to a smaller box and its first nw orbitals."""
    lo = [-((n - 1) // 2) for n in box]
    keep = np.all([(s.rp[:, a] >= lo[a]) & (s.rp[:, a] < lo[a] + box[a]) for a in range(3)], axis=0)
    nw = nw or s.nw
    return dataclasses.replace(s, nw=nw, ham=np.ascontiguousarray(s.ham[:, :nw, :nw]),
                               rp=np.ascontiguousarray(s.rp[keep]),
                               gw=np.ascontiguousarray(s.gw[:, keep][..., :nw, :nw]))


@pytest.mark.parametrize("name,nw,box,N,prec", [
    ("mini_w1", 1, (3, 3, 3), 6, "fp64"), ("mini_w1", 1, (3, 4, 4), 5, "fp32"), ("mini_w2a2", 1, (3, 3, 3), 5, "fp64"),
    ("chain_w2", 2, (3, 4, 4), 5, "fp64"), ("toy_sc", 4, (3, 3, 3), 5, "fp64"), ("mini_w8", 8, (3, 3, 3), 5, "fp64"),
    ("mini_w8", 8, (3, 4, 4), 5, "fp32"), ("toy_sc", 4, (3, 4, 4), 5, "bf16x3"), ("mini_w2a2", 2, (3, 3, 3), 5, "fp64"),
    ("mini_w4a2", 4, (3, 4, 4), 5, "fp64"), ("si_fcc", 8, (3, 3, 3), 4, "fp64"), ("si_fcc", 8, (3, 3, 3), 4, "fp32")])
def test_every_shape(torch_cuda, name, nw, box, N, prec):
    from paper_2306_16493_amd import Context
    s = cut(make_system(name), box, nw)
    eta, temps, mu = 0.05, [300.0, 600.0], s.mu_centroid
    ctx = Context(s)
    log(f"[workgroup] {name} {nw} orbitals, {s.nmodes} modes, box {box}, {N}^3 {prec}")
    g = gpu_run(ctx, ctx.params(N, mu, temps, eta, -1e3, 1e3, precision=prec))
    r = Oracle(s).run(N, mu, temps, eta, -1e3, 1e3)
    assert np.array_equal(g["state_k"], r["state_k"]) and np.array_equal(g["state_n"], r["state_n"])
    compare_rates(g, r["inv_tau"], r["tables"][0], r["state_k"], r["state_n"], tol=1e-10 if prec == "fp64" else 1e-4)
    assert g["counts"]["n_kq"] == r["n_kq"] and g["counts"]["n_terms"] == int(r["n_terms"].sum())
    ctx.close()
