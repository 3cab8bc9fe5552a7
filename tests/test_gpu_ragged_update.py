"""FP64 stages with the stored metric on x extents that the finish segments do not
divide keep the unfolded update (one rounding of q_s + c dt R at q's size): a
step is numa_stage_rhs and numa_rk_stage stage by stage, bit for bit (the same
kernels and sums, the update the same fused multiply-adds).  So does
NUMA_STAGE_GATHER at N = 5, 6 with the recomputed metric, whose element kernel
does not fold, whichever kernel a launch of its size runs."""
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# below and above the size from which the stored metric's stages take the split DSS
BOXES = [(1, (7, 3, 2)), (1, (149, 61, 3)), (2, (5, 2, 3)), (2, (109, 105, 5)), (3, (21, 2, 2)), (3, (53, 49, 5)),
         (4, (6, 4, 2)), (4, (45, 41, 5)), (5, (7, 2, 2)), (5, (46, 41, 6)), (6, (5, 2, 2)), (6, (31, 27, 3)),
         (7, (3, 2, 2)), (7, (31, 31, 4)), (8, (3, 2, 2)), (8, (29, 28, 5))]


@pytest.mark.parametrize("N,ne", BOXES)
def test_ragged_update(torch_cuda, N, ne):
    import torch
    from paper_1511_01561_amd import numa
    nx, ny, nz = ne
    wl = inputs.box_workload(nx, ny, nz, N, nx * 3.0e3, ny * 2.5e3, nz * 1.5e3, terrain=300.0)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=1)
    q0 = torch.from_numpy(inputs.random_state(g.n_unique, seed=400 + N)).cuda()
    dt = 0.02
    cases = [(numa.METRIC_STORED, m) for m in (numa.STAGE_AUTO, numa.STAGE_SPLIT, numa.STAGE_GATHER)]
    if N in (5, 6):
        cases.append((numa.METRIC_RECOMPUTE, numa.STAGE_GATHER))
    for metric, mode in cases:
        g.set_metric(metric)
        g.set_stage(mode)
        s1 = g.rk_stage(0, dt, q0, q0, g.stage_rhs(q0))
        s2 = g.rk_stage(1, dt, q0, s1, g.stage_rhs(s1))
        want = g.rk_stage(2, dt, q0, s2, g.stage_rhs(s2))
        got = g.step(q0.clone(), dt, 1)
        assert torch.equal(got.view(-1), want.view(-1)), (metric, mode)
