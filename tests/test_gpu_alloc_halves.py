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
            if budget == 8 * (cells - 1):
                assert plan.allocate_route()["route"] == ("halves" if L >= (24 if J <= 16 and cells < 16384 else 16) else "rows")
            assert np.array_equal(j.cpu().numpy(), j_ref), (kind, budget)
            assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref), (kind, budget)
            assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), (kind, budget)
    E[L // 2, J // 2] = np.inf
    j, K, off, st = plan.allocate(8 * (cells - 1), torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == ko.ERR_NONFINITE and not K.cpu().numpy().any()
    plan.close()


@pytest.mark.parametrize("cells,L", [(4225, 24), (9000, 33), (400, 64), (4200, 64)])
@pytest.mark.parametrize("scale", [1e308, 1e300, 1e-310, 1e-318])
def test_errors_at_the_ends_of_the_doubles(cells, L, scale):
    """Errors of both signs, one after the other in the layers' own order, whose sums over every second layer leave the doubles: the
    sizes are those of the sums in that order all the same (rows beyond LDS, and by the tree of segments)."""
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(cells + L)
    J = 12
    ratios = np.append(np.sort(rng.uniform(0.001, 0.99, size=J - 1)), 1.0)
    # layers that reach least first: every second one has errors below zero
    sizes = sorted(max(40, int(x)) for x in cells / L * 10.0 ** rng.uniform(-0.5, 0.9, size=L))
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    sign = np.where(np.arange(L) % 2, 1.0, -1.0)[:, None]
    E = scale * sign * (1.0 - rng.uniform(0.0, 0.8 / L, size=(L, 1)) * (Kt / np.array(sizes)[:, None]) ** rng.uniform(0.3, 1.0, size=(L, 1)) * sign)
    assert np.isfinite(E).all()
    budget = 8 * max(cells - 1, int(Kt[:, 0].sum()) + 1)
    D = 0 if cells > 4224 else cells - 1
    z = [torch.zeros(int(sum(sizes)), dtype=torch.float32, device="cuda") for _ in range(2)]
    plan = kimad.Plan(z[0], z[1], sizes, ratios.tolist(), D=D, max_budget_bytes=budget, capacity_pairs=1)
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, D)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(np.ascontiguousarray(E).reshape(-1)).cuda())
    assert int(st.item()) == st_ref == ko.OK
    assert np.array_equal(j.cpu().numpy(), j_ref)
    assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref)
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()
