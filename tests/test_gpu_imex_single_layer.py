"""One-layer meshes of many lines, which take a lane per line (imex_lines_ok):
a numa_imex_step against the oracle on sampled vertical lines, FP64 1e-12
relative max-norm per variable group; fewer lines of the same meshes take a
lane per line and layer and are in test_gpu_imex.py."""
import numpy as np
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import TOL64, Pair, assert_groups, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,N,ne", [("box", 5, (40, 34)), ("box", 8, (26, 20)), ("shell", 4, 19)])
def test_single_layer(torch_cuda, oracle_mod, kind, N, ne):
    if kind == "box":
        wl = inputs.box_workload(*ne, 1, N, ne[0] * 3.0e3, ne[1] * 3.0e3, 2.0e3, terrain=200.0)
    else:
        wl = inputs.shell_workload(ne, 1, N, H=2.0e3)
    p = Pair(wl, oracle_mod, prec_mask=5)
    assert p.o.n_horiz >= 33000
    qm, q0 = (inputs.random_state(p.nu, 450 + k) for k in (0, 1))
    lines = np.unique(np.random.default_rng(7).integers(0, p.o.n_horiz, 40))
    oa, ob = p.o.imex_step(qm, q0, 0.05, 0.05, 1, lines=lines)
    ga, gb = p.dev(qm), p.dev(q0)
    p.g.imex_step(ga, gb, 0.05, 0.05, 1)
    idx = (lines[None, :] + p.o.n_horiz * np.arange(p.o.n_levels)[:, None]).ravel()
    for name, a, b in (("q^{n+1}", p.host(gb), ob), ("filtered q^n", p.host(ga), oa)):
        assert_groups(a[:, idx], b[:, idx], TOL64, "one layer %s N=%d %s" % (kind, N, name))
