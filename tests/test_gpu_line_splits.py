"""GPU: what the launch and the index maps of the split line kernel decide,
against the FP64 oracle.

One launch for two directions of equal extended length but different node
counts, line counts that leave a last unit with one line, one, two and three
stages on one, two and four waves, the length 1125, and FC tables with fewer
and more matching points than the built-in five.

The bars are those of the length sweep: u^K to 1e-10, G and the gradients
(the latter against the oracle's adjoint of the library's own misfit) to
max(1e-10, 4 x floor), the floor being the oracle's FFT path against its
dense-matrix path; FP32 to 1e-5."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Oracle

from test_gpu_parity import TOL32, TOL64, _measured, rel, say, tol

pytestmark = pytest.mark.gpu

# (nodes along x, along y, matching points d, blend length C)
CASES = [
    (66, 65, 5, 25),      # 96, 90: two launches, odd and even line counts
    (281, 295, 5, 25),    # both 320, different extensions, one launch
    (120, 11, 5, 25),     # 150 and 36 (the latter has no split)
    (350, 33, 5, 25),     # 375: two stages with radices 15 and 25
    (216, 230, 5, 25),    # 243 and 256
    (1100, 12, 5, 25),    # 1125
    (65, 40, 3, 22),
    (160, 64, 7, 26),
]


@pytest.mark.parametrize("nx,ny,d,C", CASES)
def test_split_kernel_matches_oracle(nx, ny, d, C):
    from paper_2202_09421_amd import rte
    from paper_2202_09421_amd.fc_tables import fc_tables
    beams = [W.beam_at(0.5, 0.0, 0, 1.0, 0, (ny - 1) / (nx - 1), sigma_t=2.0, t0=0.0, sigma_x=0.2)]
    spec = W.small_problem(N=nx - 1, M=12, K=4, Ny=ny - 1, seed=nx, n_in=1.4, g=0.8, beams=beams).with_(fc_d=d, fc_C=C)
    o, od = Oracle(spec), Oracle(spec, dense_derivative=True)
    G_o, u_o, st = o.forward(keep_states=True)
    G_d, _, st_d = od.forward(keep_states=True)
    Gm = _measured(G_o, nx)
    for dtype in (torch.float64, torch.float32):
        plan = rte.Plan(spec, dtype, fc_QA=fc_tables(d, C))
        _, u = plan.forward(spec.mu_a, spec.mu_s, want_u_final=True)
        J, ga, gb, G = plan.gradient(spec.mu_a, spec.mu_s, Gm)
        torch.cuda.synchronize()
        G = G.cpu().numpy()
        src = spec.dt * (G - Gm)
        ga_o, gb_o = o.adjoint(src, st)
        ga_d, gb_d = od.adjoint(src, st_d)
        errs = dict(u=rel(u.cpu(), u_o), G=rel(G, G_o), ga=rel(ga.cpu(), ga_o), gb=rel(gb.cpu(), gb_o))
        floors = dict(u=0.0, G=rel(G_d, G_o), ga=rel(ga_d, ga_o), gb=rel(gb_d, gb_o))
        say("%dx%d d %d %s: %s floors %s" % (nx, ny, d, dtype, {k: "%.1e" % v for k, v in errs.items()},
                                             {k: "%.1e" % v for k, v in floors.items()}))
        for k, e in errs.items():
            assert e < (TOL32 if dtype == torch.float32 else (TOL64 if k == "u" else tol(floors[k]))), (k, e, floors[k])
        plan.close()
