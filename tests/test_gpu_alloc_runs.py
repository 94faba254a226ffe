"""Runs of sizes that cost the same: of equal errors the lowest member is the dynamic programme's, and so is one whose error is larger
but vanishes beside the total.  Runs of every length up to the whole grid, of members equal, a unit in the last place apart, and
further apart than the total's last place, below one another in any order that falls; against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J", [2, 3, 16, 63, 64])
@pytest.mark.parametrize("big", [0.0, 1.0, 1e6])
def test_members_of_a_run(J, big):
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(J + int(big))
    L, cells = 90, 600
    ratios = np.append(np.sort(rng.uniform(0.01, 0.99, size=J - 1)), 1.0)
    sizes = [int(x) for x in 10.0 ** rng.uniform(0.5, 4.0, size=L)]          # a cost unit is about 140 entries
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes])
    n = int(sum(sizes))
    z = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2)]
    plan = kimad.Plan(z[0], z[1], sizes, ratios.tolist(), D=cells, max_budget_bytes=8 * n, capacity_pairs=1)
    ways = []
    budget = 8 * (int(Kt[:, 0].sum()) + (n - int(Kt[:, 0].sum())) // 3)
    for turn in range(6):
        E = np.empty((L, J))
        for i in range(L):
            e = rng.uniform(0.5, 1.0) * 10.0 ** rng.uniform(-9, 0)
            for j in range(J - 1, -1, -1):
                E[i, j] = e
                step = rng.integers(0, 4)
                e = e if step == 0 else np.nextafter(e, 2.0) if step == 1 else e * (1.0 + 1e-14) if step == 2 else e * 1.01
        E[L // 2] += big                                                     # the totals' last place is that of the largest errors
        st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, cells)
        j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
        assert int(st.item()) == st_ref == ko.OK
        assert np.array_equal(j.cpu().numpy(), j_ref), turn
        ways.append(plan.allocate_route())
        assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref)
        assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    assert all(w["route"] == "tree" for w in ways)
    if J >= 16:                                          # (of two or three sizes, whole rows decide)
        assert any(w["from_left"] for w in ways)
    plan.close()
