"""The allocation of rows beyond LDS by two halves of the layers: every plan's sizes are the oracle's dynamic programme's bit for bit,
where all choices are clear and where rounding decides, at the edges of workgroups and of the longest rows, from calls in turn on
one plan."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko
from tests.test_gpu_alloc_tree import _table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,L", [(4225, 16), (4289, 17), (6144, 64), (6145, 129), (20011, 62), (131072, 16)])
@pytest.mark.parametrize("J", [5, 17, 33])
def test_sizes_are_the_oracles(cells, L, J):
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(1000 * cells + 10 * L + J)
    ratios = np.concatenate([[0.001], np.sort(rng.uniform(0.002, 0.99, size=J - 2)), [1.0]])
    sizes = [max(1, int(x)) for x in cells / L * 10.0 ** rng.uniform(-2, 0.9, size=L)]
    sizes[0] = 2 * cells                                 # (more than the rows hold)
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    n = int(sum(sizes))
    z = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2)]
    least = int(Kt[:, 0].sum())
    plan = kimad.Plan(z[0], z[1], sizes, ratios.tolist(), D=0, max_budget_bytes=8 * (cells - 1), capacity_pairs=1)
    for kind in ("falling", "ties", "noise", "tiny", "zeros", "falling"):
        E = np.ascontiguousarray(_table(rng, sizes, Kt, kind))
        table = torch.from_numpy(E.reshape(-1)).cuda()
        for budget in (8 * (cells - 1), 8 * (least + (cells - 1 - least) // 2)) if cells < 10000 else (8 * (cells - 1),):
            st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
            j, K, off, st = plan.allocate(budget, table)
            assert int(st.item()) == st_ref == ko.OK, (kind, budget)
            assert np.array_equal(j.cpu().numpy(), j_ref), (kind, budget)
            assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref), (kind, budget)
            assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), (kind, budget)
    E[L // 2, J // 2] = np.inf
    j, K, off, st = plan.allocate(8 * (cells - 1), torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == ko.ERR_NONFINITE and not K.cpu().numpy().any()
    plan.close()
