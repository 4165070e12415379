"""The device memory that a rates call takes against the least budget that it
accepts: a first call on a context allocates no more than that, and nearly all
of it, so that no budget that would do is refused.

Slack: each of some 25 buffers is rounded up to 2 MiB by the allocator.  The
kernels run once on a small grid before, so that what the runtime takes for them
itself (code, scratch of the instances that spill: 116 bytes a lane with 8 bands
and 6 modes in FP32) is there already.
"""
import gc

import numpy as np
import pytest

from gpu_helpers import log
from test_gpu_slabs import least_budget
from test_gpu_workgroup import cut
from synth import make_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,box,N,temps,prec", [
    ("si_fcc", None, 80, 1, "fp32"), ("si_fcc", None, 70, 3, "bf16x3"), ("al_fcc", None, 140, 1, "fp64"),
    ("al_fcc", None, 140, 2, "fp64"), ("al_fcc", None, 140, 1, "fp32"), ("al_fcc", None, 140, 4, "fp32"),
    ("al_fcc", (5, 5, 5), 140, 1, "fp32")])
def test_least_budget_is_what_the_call_takes(name, box, N, temps, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_16493_amd import Context
    s = make_system(name)
    s = cut(s, box) if box else s
    ks = np.array([5, 77])
    par = lambda ctx, b, N=N: ctx.params(N, s.mu_centroid, [200.0, 300.0, 400.0, 500.0][:temps], 0.02, -1e3, 1e3,
                                    precision=prec, k_subset=ks, mem_budget_bytes=b)
    probe = Context(s)
    probe.scattering_rates(par(probe, 0, 6))
    least = least_budget(lambda b: probe.scattering_rates(par(probe, b), capacity=2 * s.nw))[2]
    probe.close()
    ctx = Context(s)
    n = 2 * s.nw
    buffers = dict(k=torch.empty(n, dtype=torch.int32, device="cuda"), n=torch.empty(n, dtype=torch.int32, device="cuda"),
                   e=torch.empty(n, dtype=torch.float64, device="cuda"),
                   v=torch.empty(n, 3, dtype=torch.float64, device="cuda"),
                   it=torch.empty(temps * n, dtype=torch.float64, device="cuda"))
    gc.collect()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    res, _ = ctx.scattering_rates(par(ctx, least), capacity=n, buffers=buffers)
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0]
    log(f"[budget] {name} {N}^3 {prec}, {temps} temperatures: least {least} bytes, took {took} ({took / least:.3f})")
    assert res.counts["n_states"] == n
    assert took <= least + 25 * (2 << 20)
    assert took >= 0.95 * least
    ctx.close()
