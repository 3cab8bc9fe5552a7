"""The mass fluxes of mixed-precision shell stages are rounded to FP32 once, from
the FP64 product rho u, in the column kernel (numa_stage_rhs on these sizes) as
in the one-node-per-lane kernel (numa_rhs).  With every velocity component
c = 8 (1 + 0.49 2^-23), which FP32 rounds to 8, a flux formed from the rounded
velocity is too small by the factor 1 - 5.8e-8 at every node, and so is the mass
row; rounding the products once leaves errors of either sign, which average out
in the least-squares slope between the two (each node's is below 1e-6 of the
row's size, over more than 10^4 nodes): |slope - 1| <= 1e-8."""
import numpy as np
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,ne,nz", [(1, 30, 6), (2, 20, 5), (3, 25, 3), (4, 19, 3), (5, 18, 2), (6, 14, 3),
                                     (7, 19, 2), (8, 13, 2)])
def test_mass_flux_rounded_once(torch_cuda, N, ne, nz):
    import torch
    from paper_1511_01561_amd import numa
    wl = inputs.shell_workload(ne, nz, N, H=nz * 3.0e3)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=3)
    g.set_metric(numa.METRIC_RECOMPUTE)
    q = inputs.random_state(g.n_unique, seed=390 + N, rho_scale=0.2)
    q[1:4] = 8.0 * (1.0 + 0.49 * 2.0 ** -23)
    assert np.float32(q[1, 0]) == 8.0
    q = torch.from_numpy(q).cuda()
    want = g.dss(g.rhs(q, prec=numa.PREC_MIXED), numa.DSS_MASS).view(5, -1)[0]
    got = g.stage_rhs(q, prec=numa.PREC_MIXED).view(5, -1)[0]
    slope = float(((got - want) * want).sum() / (want * want).sum())
    assert abs(slope) <= 1e-8, slope
