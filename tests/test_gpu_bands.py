"""GPU: state rows stored in bands of 11 to 19 rows.

Row counts at the edges of the bands (less than one band, a whole number of
them, one row more), read and written by the split and by the generic line
kernel, against the FP64 oracle at the bars of the other line lengths; and the
two line kernels against each other, to the sum of their bars."""
import pytest
import torch

import workloads as W

from test_gpu_line_splits import test_split_kernel_matches_oracle as check
from test_gpu_parity import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(40, 12), (40, 15), (40, 16), (31, 26), (36, 61), (14, 46)])
def test_band_edges_match_oracle(nx, ny):
    check(nx, ny, 5, 25)


@pytest.mark.parametrize("ny", [31, 52])
def test_generic_lines_over_bands(ny):
    from paper_2202_09421_amd import rte
    spec = W.small_problem(N=39, M=16, K=4, Ny=ny - 1, seed=ny, n_in=1.4, g=0.8)
    plan = rte.Plan(spec, torch.float64)
    out = {}
    for generic in (0, 1):
        plan.set_schedule({"line_generic": generic})
        _, u = plan.forward(spec.mu_a, spec.mu_s, want_u_final=True)
        out[generic] = u.clone()
    assert rel(out[0].cpu(), out[1].cpu()) < 2e-10   # each within 1e-10 of the oracle
    plan.close()


def test_padded_rows_do_not_cross_the_static_scratch():
    """379 rows of 392 nodes: 127 MiB of forward workspace as they are, 131 MiB with 390 rows."""
    import ctypes
    from paper_2202_09421_amd import rte
    spec = W.small_problem(N=391, M=16, K=3, Ny=378, seed=2, n_in=1.4, g=0.8, n_det=8)
    plan = rte.Plan(spec, torch.float64)
    lib = rte.lib()
    lib.rte_forward_noalloc.argtypes = [ctypes.c_void_p] * 6
    lib.rte_forward_noalloc.restype = ctypes.c_int
    a, b = (torch.tensor(x, device="cuda") for x in (spec.mu_a, spec.mu_s))
    G, u = plan.forward(a, b, want_u_final=True)
    G2, u2 = torch.empty_like(G), torch.empty_like(u)
    rc = lib.rte_forward_noalloc(plan._h, a.data_ptr(), b.data_ptr(), G2.data_ptr(), u2.data_ptr(),
                                 torch.cuda.current_stream().cuda_stream)
    assert rc == 0, lib.rte_last_error().decode()
    torch.cuda.synchronize()
    assert torch.equal(G, G2) and torch.equal(u, u2)
    plan.close()
