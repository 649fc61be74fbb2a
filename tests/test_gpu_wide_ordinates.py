"""GPU: ordinate counts on both sides of four row tiles of the scattering
product (64 ordinates), where its operand is no longer held in registers, with
ragged last tiles, against the FP64 oracle at the parity bars."""
import pytest
import torch

import workloads as W
from oracle.solver import Oracle

from test_gpu_parity import TOL32, TOL64, _measured, rel, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("M", [52, 64, 68, 80, 132])
def test_ordinate_counts_match_oracle(M, dtype):
    from paper_2202_09421_amd import rte
    spec = W.small_problem(N=24, M=M, K=4, Ny=20, seed=M, n_in=1.4, g=0.9)
    o, od = Oracle(spec), Oracle(spec, dense_derivative=True)
    G_o, u_o, st = o.forward(keep_states=True)
    _, _, st_d = od.forward(keep_states=True)
    Gm = _measured(G_o, M)
    plan = rte.Plan(spec, dtype)
    _, u = plan.forward(spec.mu_a, spec.mu_s, want_u_final=True)
    J, ga, gb, G = plan.gradient(spec.mu_a, spec.mu_s, Gm)
    torch.cuda.synchronize()
    src = spec.dt * (G.cpu().numpy() - Gm)
    ga_o, gb_o = o.adjoint(src, st)
    ga_d, gb_d = od.adjoint(src, st_d)
    f32 = dtype == torch.float32
    assert rel(u.cpu(), u_o) < (TOL32 if f32 else TOL64)
    for got, ref, dense in ((ga, ga_o, ga_d), (gb, gb_o, gb_d)):
        assert rel(got.cpu(), ref) < (TOL32 if f32 else tol(rel(dense, ref)))
    plan.close()
