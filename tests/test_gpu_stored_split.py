"""The split DSS with the stored metric, which NUMA_STAGE_AUTO and
NUMA_STAGE_SPLIT take from a launch size on (these boxes are above it): the
right-hand side, SSP-RK3 steps and the in-place stages of SSP-RK(5,3) equal
NUMA_STAGE_GATHER's, one node per lane, bit for bit (the same operations per
node, the copies in the same order), on x extents that do and do not fit the
finish segments, with walls and periodic."""
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

BOXES = [(1, (149, 61, 3), False), (1, (128, 60, 4), True), (2, (108, 105, 5), False), (2, (107, 95, 5), True),
         (3, (53, 49, 5), False), (3, (64, 40, 6), True), (4, (45, 41, 5), False), (4, (44, 43, 5), True),
         (5, (46, 41, 6), False), (5, (44, 44, 6), True), (6, (31, 27, 3), False), (6, (28, 25, 4), True),
         (7, (31, 31, 4), False), (7, (32, 30, 4), True), (8, (29, 28, 5), False), (8, (28, 26, 5), True)]


@pytest.mark.parametrize("N,ne,perz", BOXES)
def test_stored_split(torch_cuda, N, ne, perz):
    import torch
    from paper_1511_01561_amd import numa
    nx, ny, nz = ne
    wl = inputs.box_workload(nx, ny, nz, N, nx * 3.0e3, ny * 2.5e3, nz * 1.5e3, terrain=0.0 if perz else 300.0,
                             periodic_z=perz)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=1)
    q = torch.from_numpy(inputs.random_state(g.n_unique, seed=430 + N, rho_scale=0.04)).cuda()
    out = {}
    for mode in (numa.STAGE_GATHER, numa.STAGE_AUTO, numa.STAGE_SPLIT):
        g.set_stage(mode)
        res = [g.stage_rhs(q)]
        for rk in (numa.RK_SSP33, numa.RK_SSP53):
            g.set_integrator(rk)
            res.append(g.step(q.clone(), 0.02, 1))
        out[mode] = res
    for mode in (numa.STAGE_AUTO, numa.STAGE_SPLIT):
        for a, b in zip(out[mode], out[numa.STAGE_GATHER]):
            assert torch.equal(a.view(-1), b.view(-1)), mode
