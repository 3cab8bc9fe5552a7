"""FP64 steps of the shell's column kernel, whose contributions off the bottom and
top levels are J w (q_s + c dt R): against numa_rhs, numa_dss and numa_rk_stage
composed stage by stage (one lane per node, nothing folded), at every order, the
wall levels by themselves.  Each stage's state agrees to the rounding of the state
(a few units of 1.1e-16 a copy) and of c dt R (the recomputed J w's mass against
the stored one's, 1e-14 of an increment below the state's size): 1e-13 of the
largest value per variable group.  A step of this size moves every group by more
than 1e-6 of it."""
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import assert_groups, group_err, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# sizes from which the column kernel runs (FP64: N <= 7)
SHELLS = [(1, 11, 4), (2, 15, 3), (3, 23, 3), (4, 19, 3), (5, 18, 2), (6, 9, 2), (7, 19, 2)]


@pytest.mark.parametrize("N,ne,nz", SHELLS)
def test_folded_step(torch_cuda, N, ne, nz):
    import torch
    from paper_1511_01561_amd import numa
    wl = inputs.shell_workload(ne, nz, N, H=nz * 3.0e3)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=1)
    g.set_metric(numa.METRIC_RECOMPUTE)
    q0 = torch.from_numpy(inputs.random_state(g.n_unique, seed=460 + N, rho_scale=1e-3)).cuda()
    dt, flags = 0.02, numa.DSS_MASS | numa.DSS_NOFLUX
    qs = q0
    for stage in range(3):
        qs = g.rk_stage(stage, dt, q0, qs, g.dss(g.rhs(qs), flags)).view(5, -1)
    want = qs.cpu().numpy()
    got = g.step(q0.clone(), dt, 1).view(5, -1).cpu().numpy()
    assert min(group_err(want, q0.cpu().numpy()).values()) > 1e-6
    nh = g.n_horiz
    for name, part in (("bottom", slice(0, nh)), ("inside", slice(nh, -nh)), ("top", slice(-nh, None))):
        assert_groups(got[:, part], want[:, part], 1e-13, "N=%d %s" % (N, name))
