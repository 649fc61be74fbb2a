"""GPU: both directions of a small grid in one launch although their extended
lengths differ, against the FP64 oracle at the bars of the other line lengths,
over lengths whose units have one, two and four waves; and a grid on either side
of the size up to which that launch is taken, bit for bit the same per source."""
import pytest
import torch

import workloads as W

from test_gpu_line_splits import test_split_kernel_matches_oracle as check

pytestmark = pytest.mark.gpu


# extended lengths: 50 48, 60 90, 81 64, 96 135, 128 256, 162 75, 216 125, 243 100, 250 54
@pytest.mark.parametrize("nx,ny", [(25, 21), (33, 65), (56, 39), (68, 110), (102, 231), (137, 49), (188, 98),
                                   (216, 75), (222, 29)])
def test_mixed_lengths_match_oracle(nx, ny):
    check(nx, ny, 5, 25)


@pytest.mark.parametrize("N,Ny", [(149, 139), (99, 59)])
def test_chunked_sources_bitwise_equal(N, Ny):
    """Eight sources at once (two launches) and one by one (one launch)."""
    from paper_2202_09421_amd import rte
    beams = []
    for k in range(8):
        b = W.beam_at(0.5, 0.0, 0, 1, 0, Ny / N, sigma_t=2.0, t0=1.0, sigma_x=0.1, tau=0.3 * k)
        b.group = k
        beams.append(b)
    spec = W.small_problem(N=N, M=32, K=4, Ny=Ny, seed=N, n_in=1.4, n_det=8).with_(beams=beams)
    out = []
    for chunk in (0, 1):
        plan = rte.Plan(spec, torch.float64, combo_chunk=chunk)
        gm = torch.zeros((plan.Nq, plan.Nd, spec.K), dtype=torch.float64, device="cuda")
        out.append([x.cpu() for x in plan.gradient(spec.mu_a, spec.mu_s, gm)])
        plan.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
