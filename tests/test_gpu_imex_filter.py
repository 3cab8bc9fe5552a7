"""The Robert-Asselin value q^n + ra (q^{n-1} - 2 q^n + q^{n+1}) of numa_imex_step
is rounded once at q's size: against the same from the step's own q^{n+1} in
extended precision, within half a unit in the last place and twice the rounding
of the bracket, which ra scales down."""
import numpy as np
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.mark.parametrize("kind,N,nz", [("box", 1, 4), ("box", 4, 3), ("box", 7, 2), ("box", 2, 33), ("shell", 3, 2),
                                       ("shell", 6, 2), ("shell", 2, 33)])
def test_filtered_level(torch_cuda, kind, N, nz):
    import torch
    from paper_1511_01561_amd import numa
    if kind == "box":
        wl = inputs.box_workload(6, 5, nz, N, 18.0e3, 15.0e3, 600.0 * nz, terrain=200.0)
    else:
        wl = inputs.shell_workload(3, nz, N, H=0.8e3 * nz)
    g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=5)
    qp, qc = (inputs.random_state(g.n_unique, 410 + k) for k in (0, 1))
    ra = 0.01
    a, b = torch.from_numpy(qp).cuda(), torch.from_numpy(qc).cuda()
    g.imex_step(a, b, 0.05, ra, 1)
    got, new = a.cpu().numpy(), b.cpu().numpy()
    p, c, n = (x.astype(np.longdouble) for x in (qp, qc, new))
    want = c + np.longdouble(ra) * (p - 2 * c + n)
    bound = 0.5 * np.spacing(np.abs(got)) + 2 * ra * U * (np.abs(p) + 2 * np.abs(c) + np.abs(n))
    bad = np.abs(got.astype(np.longdouble) - want) > bound
    assert not bad.any(), bad.mean(axis=1)
