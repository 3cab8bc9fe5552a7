"""The DSS sum of a mixed-precision box stage is FP64: numa_stage_rhs against
numa_dss of numa_rhs in the same precision.  The element kernels form the same
FP32 contributions, so the two differ by the rounding of FP64 sums of at most
eight copies, of M^-1 (the recomputed J w's mass against the stored one's,
1e-14) and of the wall projection: within 1e-13 of M^-1 sum |J w R| at every
node.  A sum of two copies in FP32 is off by up to 6e-8 of it."""
import numpy as np
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

BOXES = [(1, (70, 3, 2), False), (2, (30, 2, 3), True), (3, (21, 3, 2), False), (4, (12, 3, 2), True),
         (5, (9, 2, 2), False), (6, (5, 3, 2), False), (7, (4, 3, 2), True), (8, (3, 2, 2), False)]


def _case(N, ne, perz, metric):
    import torch
    from paper_1511_01561_amd import numa
    nx, ny, nz = ne
    wl = inputs.box_workload(nx, ny, nz, N, nx * 3.0e3, ny * 2.5e3, nz * 1.5e3, terrain=0.0 if perz else 300.0,
                             periodic_z=perz)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=3)
    g.set_metric(metric)
    q = torch.from_numpy(inputs.random_state(g.n_unique, seed=380 + N)).cuda()
    c = g.rhs(q, prec=numa.PREC_MIXED).view(5, -1)
    want = g.dss(c, numa.DSS_MASS | numa.DSS_NOFLUX).cpu().numpy()
    scale = g.dss(c.abs(), numa.DSS_MASS).cpu().numpy()
    scale[1:4] = scale[1:4].sum(axis=0)  # the projection mixes the components
    return g, q, want, scale


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("N,ne,perz", BOXES)
def test_gather_sums(torch_cuda, N, ne, perz, metric):
    from paper_1511_01561_amd import numa
    g, q, want, scale = _case(N, ne, perz, metric)
    for mode in (numa.STAGE_AUTO, numa.STAGE_GATHER):
        g.set_stage(mode)
        r = g.stage_rhs(q, prec=numa.PREC_MIXED).cpu().numpy()
        assert (np.abs(r - want) / scale).max() <= 1e-13, mode


@pytest.mark.parametrize("N,ne,perz", BOXES[:4])
def test_split_sums(torch_cuda, N, ne, perz):
    """The split DSS stores a pair inside a run of a face row as one FP32
    value; every other sum (the run-interior nodes' pairs, the pairs across run
    starts, here all of x = 0, and the sums over y and z) is FP64."""
    from paper_1511_01561_amd import numa
    g, q, want, scale = _case(N, ne, perz, numa.METRIC_RECOMPUTE)
    g.set_stage(numa.STAGE_SPLIT)
    r = g.stage_rhs(q, prec=numa.PREC_MIXED).cpu().numpy()
    gi = np.arange(g.n_unique) % (ne[0] * N)
    gj = np.arange(g.n_unique) // (ne[0] * N) % (ne[1] * N)
    gk = np.arange(g.n_unique) // g.n_horiz
    pair = (gi % N == 0) & (gi > 0) & ((gj % N == 0) | (gk % N == 0))
    # rho' has other contributions here: the kernel forms rho u from the FP32 velocity
    assert (np.abs(r - want) / scale)[1:, ~pair].max() <= 1e-13
