"""GPU: unequal extended lengths on both sides of the limit of the combined launch.

Lengths that use different numbers of waves share a launch up to 2048 blocks;
blocks of the shorter lines then hold a wave without work.  Two sources at once
exceed that and take two launches, one source does not: the same bits per
source, whatever the launch."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _units(lines):
    pairs = (lines + 1) // 2
    return pairs + pairs % 2


# extended lengths 216 (two waves a unit) and 72 (one); 41 lines: one without a partner
@pytest.mark.parametrize("nx,ny", [(180, 40), (41, 180)])
@pytest.mark.parametrize("f32", [0, 1])
def test_different_wave_counts_bitwise_equal(nx, ny, f32):
    from paper_2202_09421_amd import rte
    M = 64
    blocks = (_units(ny) + _units(nx) + 15) // 16 * 16 * (M // 4)
    assert blocks <= 2048 < 2 * blocks
    beams = []
    for k in range(2):
        b = W.beam_at(0.5, 0.0, 0, 1, 0, (ny - 1) / (nx - 1), sigma_t=2.0, t0=1.0, sigma_x=0.1, tau=0.3 * k)
        b.group = k
        beams.append(b)
    spec = W.small_problem(N=nx - 1, Ny=ny - 1, M=M, K=4, seed=nx, n_in=1.4, n_det=8).with_(beams=beams)
    out = []
    for chunk in (0, 1):
        plan = rte.Plan(spec, torch.float32 if f32 else torch.float64, combo_chunk=chunk)
        assert {plan.Np_x, plan.Np_y} == {216, 72}
        gm = torch.zeros((plan.Nq, plan.Nd, spec.K), dtype=torch.float64, device="cuda")
        out.append([x.cpu() for x in plan.gradient(spec.mu_a, spec.mu_s, gm)])
        plan.close()
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)
