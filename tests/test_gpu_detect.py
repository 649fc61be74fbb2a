"""GPU: the detector kernel at the edges of its blocks (2 time levels x 4
detectors, 256 boundary positions) against the oracle's traces: u^K to 1e-10,
G to max(1e-10, 4 x floor), the floor being the oracle's FFT path against its
dense-matrix path."""
import pytest
import torch

import workloads as W
from oracle.solver import Oracle

from test_gpu_parity import rel, say, tol

pytestmark = pytest.mark.gpu


# 4 x max(nodes per side) positions: 60, 256, 260, 600
@pytest.mark.parametrize("N,Ny,n_det,K", [(14, 10, 1, 1), (14, 10, 5, 3), (63, 10, 4, 2), (64, 12, 3, 5), (149, 10, 9, 4)])
def test_traces_match_oracle(N, Ny, n_det, K):
    from paper_2202_09421_amd import rte
    beams = [W.beam_at(0.5, 0.0, 0, 1.0, 0, Ny / N, sigma_t=2.0, t0=0.0, sigma_x=0.3, group=g) for g in (0, 1)]
    spec = W.small_problem(N=N, Ny=Ny, M=8, K=K, seed=N + n_det, n_in=1.4, n_det=n_det, beams=beams)
    G_o, _, _ = Oracle(spec).forward()
    G_d, _, _ = Oracle(spec, dense_derivative=True).forward()
    for chunk in (0, 1):
        plan = rte.Plan(spec, torch.float64, combo_chunk=chunk)
        G = plan.forward(spec.mu_a, spec.mu_s).cpu().numpy()
        e, floor = rel(G, G_o), rel(G_d, G_o)
        say("N %d Ny %d Nd %d K %d chunk %d: G %.1e floor %.1e" % (N, Ny, n_det, K, chunk, e, floor))
        assert G.shape == (2, n_det, K) and e < tol(floor)
        plan.close()
