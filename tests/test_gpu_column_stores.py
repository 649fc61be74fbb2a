"""GPU: FP32 plans on both sides of the size from which column results are
stored without the non-temporal hint (64 MiB a source), against the FP64 plan
of the same problem at the FP32 parity bar."""
import pytest
import torch

import workloads as W

from test_gpu_parity import TOL32, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [500, 520])
def test_column_stores(N):
    from paper_2202_09421_amd import rte
    spec = W.small_problem(N=N, M=64, K=3, seed=N, n_in=1.4, g=0.8, n_det=8)
    out = {}
    for dtype in (torch.float64, torch.float32):
        plan = rte.Plan(spec, dtype, ckpt_every=2)
        _, u = plan.forward(spec.mu_a, spec.mu_s, want_u_final=True)
        gm = torch.zeros((plan.Nq, plan.Nd, spec.K), dtype=torch.float64, device="cuda")
        _, ga, gb, _ = plan.gradient(spec.mu_a, spec.mu_s, gm)
        out[dtype] = [x.double().cpu() for x in (u, ga, gb)]
        plan.close()
    for a, b in zip(out[torch.float32], out[torch.float64]):
        assert rel(a, b) < TOL32
