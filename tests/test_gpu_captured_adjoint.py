"""GPU: a recorded rte_adjoint of a checkpointed forward.

A recording is launched with other cotangents, after other calls on the same
workspace, and before eager adjoints of the same forward.  The stored states
are then those of the segment, or of the chunk of sources, that the last of
these calls left there, which the host cannot know; every result must still
have the bits of a plan that keeps every state and is called eagerly."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

K = 8


def _spec():
    beams = [W.beam_at(0.5, 0.0, 0, 1.0, 0, 1.0, sigma_t=2.0, t0=0.0, sigma_x=0.2, group=0),
             W.beam_at(0.0, 0.5, 0, 1.0, 0, 1.0, sigma_t=2.0, t0=0.5, sigma_x=0.2, group=1)]
    return W.small_problem(N=18, M=12, K=K, seed=71, n_in=1.4, g=0.8, beams=beams)


def _record(call):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = call()
    return g, out


@pytest.mark.parametrize("ckpt,chunk", [(1, 0), (2, 0), (3, 0), (5, 0), (K - 1, 0), (K, 0), (0, 1), (3, 1), (K, 1)])
def test_recorded_adjoint_is_idempotent(ckpt, chunk):
    from paper_2202_09421_amd import rte
    spec = _spec()
    a, b = (torch.tensor(x, device="cuda") for x in (spec.mu_a, spec.mu_s))
    rng = np.random.default_rng(ckpt)
    cot = [torch.tensor(1e-3 * rng.standard_normal((2, len(spec.detectors), K)), device="cuda") for _ in range(3)]

    ref_plan = rte.Plan(spec, torch.float64)
    ref_plan.forward(a, b, save_states=True)
    ref = [[x.clone() for x in ref_plan.adjoint(g, a, b)] for g in cot]

    plan = rte.Plan(spec, torch.float64, ckpt_every=ckpt, combo_chunk=chunk)
    bar = torch.empty_like(cot[0])
    gm = torch.zeros_like(bar)
    plan.gradient(a, b, gm)
    grad, _ = _record(lambda: plan.gradient(a, b, gm))
    plan.forward(a, b, save_states=True)
    adj, out = _record(lambda: plan.adjoint(bar, a, b))

    def same(got, k, what):
        torch.cuda.synchronize()
        for x, y in zip(got, ref[k]):
            assert torch.equal(x, y), (ckpt, chunk, what, k)

    for k in (0, 1, 2):              # replays with other cotangents
        bar.copy_(cot[k])
        adj.replay()
        same(out, k, "replay")
    same(plan.adjoint(cot[1], a, b), 1, "eager after replay")
    bar.copy_(cot[2])
    adj.replay()
    same(out, 2, "replay after eager")
    plan.forward(a, b, save_states=True)
    adj.replay()
    same(plan.adjoint(cot[0], a, b), 0, "eager after forward and replay")
    plan.forward(a, b, save_states=True)
    grad.replay()
    same(plan.adjoint(cot[1], a, b), 1, "eager after a recorded gradient")
    ref_plan.close()
    plan.close()
