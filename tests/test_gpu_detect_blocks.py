"""GPU: more detector outputs than one launch has blocks for.

The detector kernel forms 2 time levels x 4 detectors with 256 threads, and a
launch holds 2^32 threads along x, so 2^27 outputs of a source were the limit.
Every trace must have the bits it has in a solve with few detectors (a
trace's sum does not depend on the block that forms it)."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def test_more_outputs_than_blocks():
    from paper_2202_09421_amd import rte
    K, Nd = 65602, 2050
    assert (K // 2) * (Nd // 4) * 256 > 2 ** 32
    spec = W.small_problem(N=10, M=4, K=K, Ny=9, seed=5, n_det=Nd)
    plan = rte.Plan(spec, torch.float64)
    G = plan.forward(spec.mu_a, spec.mu_s)
    for part in (slice(0, 5), slice(1021, 1028), slice(Nd - 3, Nd)):
        few = rte.Plan(spec.with_(detectors=spec.detectors[part]), torch.float64)
        assert torch.equal(G[:, part], few.forward(spec.mu_a, spec.mu_s)), part
        few.close()
    assert bool(torch.isfinite(G).all()) and float(G.abs().max()) > 0
    plan.close()
