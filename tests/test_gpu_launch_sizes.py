"""Work of more threads than a launch holds (2^32 along x; some larger launches
are not refused but wrap and run a part)."""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import log, gpu_run
from test_gpu_workgroup import cut
from synth import make_system
from synth.systems import _draw_g, lattice_block

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_state_operand_of_the_bf16_transform(torch_cuda):
    """One batch of 81^3 states of one band, 2 x 4096 operand values each:
    4.35e9 values, a thread each.  Rates of the last k points against a call
    with those alone, 1e-12 as for other slabs, and against FP64, 1e-4.  The
    bands are stretched to some 1e4 eV, so that few terms are kept: a state
    still scatters to -k (time reversal)."""
    from paper_2306_16493_amd import Context
    s = make_system("mini_w1")
    re = lattice_block(16)
    gw = _draw_g(np.random.default_rng(5), s.lattice, re, s.rp, 3, 1)
    s = dataclasses.replace(s, re=re, gw=gw, ham=s.ham * 1e4)
    N, temps, eta = 81, [300.0], 0.02
    ctx = Context(s)
    ctx.set_profiling(True)
    full = gpu_run(ctx, ctx.params(N, 0.0, temps, eta, -1e9, 1e9, precision="bf16x3"))
    assert ctx.stage_times()["xform_launches"] == 1 and full["counts"]["n_states"] * 8192 > 1 << 32
    ks = np.concatenate([np.arange(0, 40), N ** 3 // 2 + np.arange(0, 40), np.arange(N ** 3 - 100, N ** 3)])
    few = gpu_run(ctx, ctx.params(N, 0.0, temps, eta, -1e9, 1e9, precision="bf16x3", k_subset=ks))
    ref = gpu_run(ctx, ctx.params(N, 0.0, temps, eta, -1e9, 1e9, k_subset=ks))
    assert np.array_equal(full["state_k"][ks], few["state_k"])
    scatters = ref["inv_tau"][0] > 0.0
    log(f"[launch] {full['counts']['n_states']} states, {scatters.sum()} of {len(ks)} compared scatter")
    assert scatters.sum() > 100 and np.isfinite(full["inv_tau"]).all()
    assert np.allclose(full["inv_tau"][0][ks], few["inv_tau"][0], rtol=1e-12, atol=0.0)
    assert np.allclose(full["inv_tau"][0][ks], ref["inv_tau"][0], rtol=1e-4, atol=0.0)
    ctx.close()


def test_conversion_walks_over_its_elements(torch_cuda):
    """FP32 rotation tables of the workgroup form, 3.5e6 elements: more than one
    step of the conversion's grid.  FP32 against FP64, 1e-4."""
    from paper_2306_16493_amd import Context
    s = cut(make_system("toy_sc"), (3, 3, 3))
    N = 60
    ks = np.array([0, 1000, N ** 3 - 1])
    ctx = Context(s)
    f32, f64 = (gpu_run(ctx, ctx.params(N, s.mu_centroid, [300.0], 0.05, -1e3, 1e3, precision=p, k_subset=ks))
                for p in ("fp32", "fp64"))
    assert np.allclose(f32["inv_tau"], f64["inv_tau"], rtol=1e-4, atol=0.0)
    ctx.close()
