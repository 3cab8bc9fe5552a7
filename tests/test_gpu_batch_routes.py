"""A batch whose NUMA_STAGE_AUTO items together take another route than each
alone (auto_route, auto_route_stored: each item is below the order's line, their
sum above it) gives each item the result of numa_step on it alone, bit for bit:
one node per lane alone against the column gather, the streaming gather, the
split DSS and its line kernel in the batch, and the split's line kernel alone
(rows_below) against its column kernel in the batch."""
import pytest

from paper_1511_01561_amd import inputs
from test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# precision, metric, order, item sizes (repeated to the count given), steps
FP64, MIXED, STORED, RECOMPUTE = 0, 1, 0, 1
CASES = [
    (FP64, RECOMPUTE, 1, [(40, 8, 8), (17, 15, 9), (24, 20, 6)], 4),         # column gather
    (FP64, RECOMPUTE, 2, [(12, 11, 10), (21, 12, 9), (16, 16, 8)], 4),       # column gather
    (FP64, RECOMPUTE, 3, [(16, 11, 12), (13, 13, 12), (21, 10, 9)], 4),      # column gather
    (FP64, RECOMPUTE, 3, [(16, 12, 14), (13, 15, 14), (21, 12, 11)], 6),     # split
    (FP64, RECOMPUTE, 4, [(20, 13, 10), (21, 12, 9), (16, 16, 10)], 5),      # split
    (FP64, RECOMPUTE, 5, [(20, 13, 9), (21, 12, 9), (17, 14, 10)], 5),       # split, lines
    (FP64, RECOMPUTE, 6, [(12, 7, 7), (11, 7, 8), (9, 9, 8)], 3),            # split, lines
    (FP64, RECOMPUTE, 5, [(40, 34, 8), (37, 30, 10)], 2),                    # lines alone, columns
    (FP64, RECOMPUTE, 6, [(29, 31, 10), (32, 28, 9)], 2),                    # lines alone, columns
    (FP64, RECOMPUTE, 7, [(12, 9, 9), (11, 10, 9), (14, 8, 8)], 4),          # split
    (FP64, RECOMPUTE, 8, [(12, 8, 8), (11, 8, 9), (10, 9, 8)], 4),           # split
    (FP64, STORED, 4, [(20, 13, 9), (16, 16, 9), (24, 10, 9)], 4),           # split
    (FP64, STORED, 6, [(12, 7, 7), (8, 9, 8), (16, 6, 6)], 4),               # split, lines
    (FP64, STORED, 5, [(20, 13, 9), (16, 16, 9), (24, 10, 10)], 4),          # split
    (FP64, STORED, 6, [(24, 24, 8), (28, 21, 8)], 3),                        # lines alone, columns
    (MIXED, RECOMPUTE, 4, [(20, 13, 4), (12, 12, 8), (16, 9, 8)], 5),        # column gather
    (MIXED, RECOMPUTE, 6, [(12, 8, 8), (8, 11, 9), (16, 7, 7)], 4),          # streaming gather
]


@pytest.mark.parametrize("prec,metric,N,sizes,count", CASES)
def test_batch_across_a_line(torch_cuda, prec, metric, N, sizes, count):
    import torch
    from paper_1511_01561_amd import numa
    items, alone = [], []
    for k in range(count):
        nx, ny, nz = sizes[k % len(sizes)]
        wl = inputs.box_workload(nx, ny, nz, N, nx * 3.0e3, ny * 2.5e3, nz * 1.5e3, terrain=300.0)
        g = numa.Mesh(wl["mesh"], wl["phys"], prec_mask=3)
        g.set_metric(metric)
        q = torch.from_numpy(inputs.random_state(g.n_unique, seed=440 + 10 * N + k, rho_scale=0.04)).cuda()
        alone.append(q.clone())
        items.append((g, q, numa.alloc_scratch(g, prec), 0.02 + 0.002 * k))
    numa.step_batch(items, 2, prec)
    for (g, q, _, dt), a in zip(items, alone):
        g.step(a, dt, 2, prec=prec)
        assert torch.isfinite(q).all() and torch.equal(q, a)
