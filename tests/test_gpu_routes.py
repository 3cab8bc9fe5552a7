"""The routes of a box stage (NUMA_STAGE_AUTO picks by the size of a launch):
one node per lane with the gather DSS, the column kernels with the gather
DSS, and the split DSS.  Where the route may depend on what a solve is batched
with, the routes give the same result bit for bit, on any x extent; against
the oracle within 1e-12 (FP64) and 1e-5 (mixed), relative max-norm per
variable group, on states on both sides of the equation of state's series
(|x| < 1/64)."""
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import TOL64, TOLMIX, Pair, assert_groups, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# x extents below, between and above the finish segments (4, 8, 16, 64 elements)
# and the runs of the column kernels, a partly empty last segment among them
CASES = [(1, (70, 3, 2), False), (1, (5, 2, 3), True), (2, (15, 3, 2), False), (2, (3, 2, 2), True),
         (3, (21, 2, 2), False), (3, (7, 3, 2), True), (4, (11, 3, 2), False), (4, (6, 2, 3), True),
         (5, (9, 2, 2), False), (6, (5, 3, 2), False), (7, (5, 2, 2), False), (8, (3, 2, 2), True)]


def _pair(N, ne, perz, oracle_mod):
    nx, ny, nz = ne
    wl = inputs.box_workload(nx, ny, nz, N, nx * 3.0e3, ny * 2.5e3, nz * 1.5e3, terrain=300.0,
                             bubble_centre=(nx * 1.5e3, ny * 1.25e3, 1.5e3), bubble_radius=3.0e3, periodic_z=perz)
    return Pair(wl, oracle_mod)


@pytest.mark.parametrize("metric", ["stored", "recompute"])
@pytest.mark.parametrize("N,ne,perz", CASES)
def test_routes_agree(torch_cuda, oracle_mod, N, ne, perz, metric):
    import torch
    from paper_1511_01561_amd import numa
    p = _pair(N, ne, perz, oracle_mod)
    p.g.set_metric(numa.METRIC_RECOMPUTE if metric == "recompute" else numa.METRIC_STORED)
    q = inputs.random_state(p.nu, seed=300 + N, rho_scale=0.04)
    assert (abs(q[0]) > 0.02).any()  # beyond the series with rho_bar of order one
    Ro = p.o.dss(p.o.rhs(q), 3)
    for prec, tol, others in ((numa.PREC_FP64, TOL64, (numa.STAGE_SPLIT,) + ((numa.STAGE_GATHER,) if N <= 4 else ())),
                              (numa.PREC_MIXED, TOLMIX, (numa.STAGE_GATHER,))):
        out = {}
        for mode in (numa.STAGE_AUTO,) + others:
            p.g.set_stage(mode)
            r = p.g.stage_rhs(p.dev(q), prec=prec)
            s = p.dev(q)
            p.g.step(s, 0.02, 2, prec=prec)
            out[mode] = (r, s)
        assert_groups(p.host(out[numa.STAGE_AUTO][0]), Ro, tol, "N=%d ne=%s prec=%d" % (N, ne, prec))
        for mode in others:
            for a, b in zip(out[numa.STAGE_AUTO], out[mode]):
                assert torch.equal(a, b), (prec, mode)


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("N,ne", [(3, (5, 3, 2)), (4, (3, 3, 3)), (6, (7, 2, 2))])
def test_filter_routes_agree(torch_cuda, oracle_mod, N, ne, metric):
    import torch
    from paper_1511_01561_amd import numa
    p = _pair(N, ne, False, oracle_mod)
    p.g.set_metric(metric)
    q = inputs.random_state(p.nu, seed=320 + N)
    out = []
    for mode in (numa.STAGE_AUTO, numa.STAGE_SPLIT):
        p.g.set_stage(mode)
        out.append(p.g.filter(p.dev(q), 12.0, 1))
    assert torch.equal(*out)
    assert_groups(p.host(out[0]), p.o.filter(q, 12.0, 1), TOL64, "filter N=%d ne=%s" % (N, ne))
