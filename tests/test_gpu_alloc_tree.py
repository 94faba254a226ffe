"""The allocation by a tree of segments: every plan's sizes are the oracle's dynamic programme's bit for bit, where all choices
are clear and where rounding decides (ties, errors that vanish beside the total), with layers that have no choice of cost, at the
edges of rows and segments, from calls in turn on one plan."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko

pytestmark = pytest.mark.gpu


def _table(rng, sizes, Kt, kind):
    n = np.array(sizes, dtype=np.float64)[:, None]
    E = 10.0 ** rng.uniform(-6, 2, size=(len(sizes), 1)) * (1.0 - Kt / n) ** rng.uniform(0.5, 6.0, size=(len(sizes), 1))
    if kind == "noise":
        E = rng.random(E.shape) - 0.3                    # neither falling nor convex, negative entries
    elif kind == "ties":
        E = np.round(4.0 * E / np.maximum(E.max(axis=1, keepdims=True), 1e-300))           # small whole numbers in every layer
    elif kind == "tiny":
        E *= 10.0 ** -rng.integers(0, 20, size=(len(sizes), 1)).astype(np.float64)       # errors below a unit in the total's last place
    elif kind == "zeros":
        E[rng.random(len(sizes)) < 0.5] = 0.0
        E[:, 1::3] = E[:, ::3][:, :E[:, 1::3].shape[1]]  # equal neighbours
    return E


@pytest.mark.parametrize("cells,L", [(90, 60), (64, 61), (90, 64), (66, 65), (575, 64), (576, 60), (1000, 60), (1023, 97), (1024, 192), (1025, 193), (1024, 1024), (1537, 24), (2049, 25),
                                     (4223, 64), (4224, 48), (4224, 300), (1536, 1024)])
@pytest.mark.parametrize("J", [2, 17, 64])
def test_sizes_are_the_oracles(cells, L, J):
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(1000 * cells + 10 * L + J)
    # (the cheapest sizes are few, so that most budgets have room for them)
    ratios = np.concatenate([rng.uniform(0.001, 0.02, size=1), np.sort(rng.uniform(0.02, 0.99, size=J - 2)), [1.0]])
    # sizes from a fraction of a cost unit (no choice) to much of the row
    sizes = [max(1, int(x)) for x in 3000.0 * 10.0 ** rng.uniform(-3, 1.5, size=L)]
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    n = int(sum(sizes))
    z = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2)]
    least = int(Kt[:, 0].sum())
    most = max(8 * n, 8 * (cells - 1))
    plan = kimad.Plan(z[0], z[1], sizes, ratios.tolist(), D=cells - 1, max_budget_bytes=most, capacity_pairs=1)
    # whole cost units, so that the rows have exactly this many cells; and too little for the cheapest
    budgets = [8 * (cells - 1) * max(1, (least + int(f * (n - least))) // (cells - 1)) for f in (0.02, 0.3)] + [8 * max(1, least // 3)]
    way = "tree" if L >= (24 if cells >= 1537 else 60 if cells >= 576 else 64) else "rows"
    for kind in ("falling", "ties", "noise", "tiny", "zeros", "falling"):
        E = np.ascontiguousarray(_table(rng, sizes, Kt, kind))
        table = torch.from_numpy(E.reshape(-1)).cuda()
        for budget in budgets if cells * L * J < 4e6 else budgets[1:2]:
            st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, cells - 1)
            j, K, off, st = plan.allocate(budget, table)
            assert int(st.item()) == st_ref, (kind, budget)
            assert budget == budgets[2] or plan.allocate_route()["route"] == way
            if st_ref != ko.OK:
                assert not K.cpu().numpy().any() and not off.cpu().numpy().any()
                continue
            assert np.array_equal(j.cpu().numpy(), j_ref), (kind, budget)
            assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref), (kind, budget)
            assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), (kind, budget)
    E[L // 2, J // 2] = np.nan
    j, K, off, st = plan.allocate(budgets[1], torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == ko.ERR_NONFINITE and not K.cpu().numpy().any()
    plan.close()


def _rising_within_runs(cells, L, J, seed):
    """Sizes of which many cost the same, errors that fall from cost to cost and, at one cost, in no order: layers keep several entries
    of one cost, the later ones of less error."""
    rng = np.random.default_rng(seed)
    ratios = np.append(np.sort(rng.uniform(0.001, 0.99, size=J - 1)), 1.0)
    sizes = [int(x) for x in 10.0 ** rng.uniform(2.5, 4.2, size=L)]
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes])
    n = int(sum(sizes))
    budget = 8 * (int(Kt[:, 0].sum()) + n // 4)
    E = (1.0 - Kt / np.array(sizes)[:, None]) ** 2 + 0.2 * rng.random(Kt.shape)
    E *= 10.0 ** rng.uniform(-3, 0, size=(L, 1))
    unit = -(-(budget // 8) // (cells - 1))
    w = -(-Kt // unit)
    pairs = 0
    for i in range(L):                                   # (kept entries of a cost that has another one)
        least, last = np.inf, -1
        for j in range(J):
            if j + 1 < J and w[i, j + 1] == w[i, j] and E[i, j + 1] <= E[i, j]:
                continue                                 # not the last of its run
            pairs += int(E[i, j] < least and last == w[i, j])
            if E[i, j] < least:
                least, last = E[i, j], w[i, j]
    assert pairs > L                                     # (a layer of them is a segment's first somewhere)
    return ratios, sizes, Kt, E, budget


@pytest.mark.parametrize("cells,L,J", [(200, 64, 33), (1000, 96, 64), (1600, 128, 64), (4200, 300, 64)])
def test_entries_of_equal_costs(cells, L, J):
    import torch
    import paper_2312_08053_amd as kimad
    ratios, sizes, Kt, E, budget = _rising_within_runs(cells, L, J, cells + L)
    z = [torch.zeros(int(sum(sizes)), dtype=torch.float32, device="cuda") for _ in range(2)]
    plan = kimad.Plan(z[0], z[1], sizes, ratios.tolist(), D=cells - 1, max_budget_bytes=budget, capacity_pairs=1)
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, cells - 1)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == st_ref == ko.OK
    assert np.array_equal(j.cpu().numpy(), j_ref)
    assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref)
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()
