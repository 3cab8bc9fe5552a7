"""numa_dss for any number of variables: one per lane, or up to five per lane on
large shells.  Unweighted sums equal the gather map's, copies in ascending
order, bit for bit; weighted and projected ones each component's own weighted
sum, bit for bit off the walls and within 1e-14 of the largest on them."""
import numpy as np
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _mesh(kind, N, ne):
    from paper_1511_01561_amd import numa
    if kind == "box":
        wl = inputs.box_workload(*ne, N, ne[0] * 3.0e3, ne[1] * 2.5e3, ne[2] * 1.5e3, terrain=300.0)
    else:
        wl = inputs.shell_workload(ne[0], ne[1], N, H=ne[1] * 3.0e3)
    return numa.Mesh(wl["mesh"], wl["phys"], prec_mask=1)


# shells on both sides of 300,000 element-local nodes
MESHES = [("box", 2, (3, 2, 2)), ("box", 5, (4, 3, 2)), ("box", 8, (2, 3, 1)), ("shell", 4, (3, 2)), ("shell", 1, (80, 1)),
          ("shell", 5, (16, 1)), ("shell", 8, (7, 2))]


@pytest.mark.parametrize("kind,N,ne", MESHES)
def test_dss_variables(torch_cuda, kind, N, ne):
    import torch
    from paper_1511_01561_amd import numa
    g = _mesh(kind, N, ne)
    G = g.gather_map().reshape(-1)
    for nvar in (1, 2, 3, 4, 5, 6, 9, 11):
        C = np.random.default_rng(420 + nvar).standard_normal((nvar, g.n_local))
        want = np.zeros((nvar, g.n_unique))
        for v in range(nvar):
            np.add.at(want[v], G, C[v])
        dev = torch.from_numpy(C).cuda()
        assert np.array_equal(g.dss(dev, 0).cpu().numpy(), want), nvar
        mass = g.dss(dev, numa.DSS_MASS).cpu().numpy()
        one = g.dss(dev[nvar - 1:], numa.DSS_MASS).cpu().numpy()
        assert np.array_equal(mass[nvar - 1:], one), nvar
    r = g.dss(dev[:5].contiguous(), numa.DSS_MASS | numa.DSS_NOFLUX).cpu().numpy()
    nh = g.n_horiz
    assert np.array_equal(r[:, nh:-nh], mass[:5, nh:-nh]) and np.array_equal(r[[0, 4]], mass[[0, 4]])
    if kind == "shell":  # the wall normal is radial
        x = g.export(numa.FIELD_COORDS).cpu().numpy()
        n = x / np.sqrt((x * x).sum(0))
        for wall in (slice(0, nh), slice(-nh, None)):
            dn = (r[1:4, wall] * n[:, wall]).sum(0)
            t = mass[1:4, wall] - (mass[1:4, wall] * n[:, wall]).sum(0) * n[:, wall]
            assert np.abs(dn).max() <= 1e-14 * np.abs(mass[1:4]).max()
            assert np.abs(r[1:4, wall] - t).max() <= 1e-14 * np.abs(mass[1:4]).max()


def test_dss_more_variables_than_one_launch(torch_cuda):
    """2^24 - 1 workgroups to a launch: variables on both sides of the next."""
    import torch
    g = _mesh("box", 1, (2, 2, 1))
    nvar = (1 << 24) + 40
    dev = torch.rand((nvar, g.n_local), dtype=torch.float64, device="cuda")
    out = g.dss(dev, 0)
    G = g.gather_map().reshape(-1)
    pick = [0, 1, (1 << 24) - 3, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, nvar - 1]
    C = dev[pick].cpu().numpy()
    want = np.zeros((len(pick), g.n_unique))
    for v in range(len(pick)):
        np.add.at(want[v], G, C[v])
    assert np.array_equal(out[pick].cpu().numpy(), want)
