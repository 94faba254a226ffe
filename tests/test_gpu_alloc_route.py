"""Which way an allocation goes, and what decides it: by the tree of segments and by halves the sizes are there where every choice is
clear, and whole rows decide where equal totals leave a choice to rounding, and only there; calls of other plans in between, and
calls in turn on one plan, report what they did themselves.  The sizes are the oracle's throughout."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko

pytestmark = pytest.mark.gpu

TREE = [(300, 64, 16), (1000, 62, 50), (1024, 200, 33), (1025, 70, 5), (1537, 24, 64), (4097, 148, 64), (4224, 300, 16)]
HALVES = [(4225, 24, 5), (4225, 16, 17), (9000, 40, 32), (16384, 16, 16), (20011, 62, 64)]


def _case(cells, L, J, alike):
    """Sizes and errors of layers that differ in scale by no more than a hundred, or (`alike`) are all the same."""
    rng = np.random.default_rng(cells + 10 * L + J)
    ratios = np.concatenate([[0.001], np.sort(rng.uniform(0.002, 0.99, size=J - 2)), [1.0]])     # (the cheapest sizes always fit)
    lo = max(60, 4 * cells // L)
    sizes = [lo + 17] * L if alike else [int(x) for x in rng.integers(lo, 4 * lo, size=L)]
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    n = np.array(sizes, dtype=np.float64)[:, None]
    E = 10.0 ** rng.uniform(-1, 1, size=(L, 1)) * (1.0 - Kt / n) ** rng.uniform(1.0, 4.0, size=(L, 1))
    if alike:
        E[:] = E[0]
    D = cells - 1 if cells <= 4224 else 0
    pairs = cells - 1 if D == 0 else (cells - 1) * max(1, int(0.3 * sum(sizes)) // (cells - 1))
    return ratios, sizes, Kt, np.ascontiguousarray(E), 8 * pairs, D


def _plan(sizes, ratios, D, budget, flags=0):
    import torch
    import paper_2312_08053_amd as kimad
    z = [torch.zeros(int(sum(sizes)), dtype=torch.float32, device="cuda") for _ in range(2)]
    return kimad.Plan(z[0], z[1], list(sizes), list(ratios), D=D, max_budget_bytes=budget, cfg_flags=flags, capacity_pairs=1)


def _allocate(plan, E, Kt, budget, D):
    import torch
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, D)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == st_ref == ko.OK
    assert np.array_equal(j.cpu().numpy(), j_ref)
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    return plan.allocate_route()


@pytest.mark.parametrize("cells,L,J", TREE + HALVES)
def test_clear_choices_need_no_whole_rows_and_ties_do(cells, L, J):
    name = "halves" if cells > 4224 else "tree"
    ratios, sizes, Kt, E, budget, D = _case(cells, L, J, False)
    plan = _plan(sizes, ratios, D, budget)
    assert plan.allocate_route() == dict(route="none", rows_decided=False, from_left=False, at_once=False)
    clear = _allocate(plan, E, Kt, budget, D)
    assert clear["route"] == name and not clear["rows_decided"], clear
    assert not any(plan.allocate_diagnostics().values())
    if L <= 1024 and cells <= 4224:
        banded = _plan(sizes, ratios, D, budget, flags=4)
        assert _allocate(banded, E, Kt, budget, D)["route"] == "band" and banded.allocate_diagnostics()["max_band"] > 0
        banded.close()
    rows = _plan(sizes, ratios, D, budget, flags=2)
    assert _allocate(rows, E, Kt, budget, D) == dict(route="rows", rows_decided=False, from_left=False, at_once=False)
    rows.close()
    assert plan.allocate_route() == clear                 # (other plans' calls are not this one's)
    plan.close()
    ratios, sizes, Kt, E, budget, D = _case(cells, L, J, True)
    plan = _plan(sizes, ratios, D, budget)
    for _ in range(2):
        tied = _allocate(plan, E, Kt, budget, D)
        assert tied == dict(route=name, rows_decided=True, from_left=False, at_once=False), tied
    assert not any(plan.allocate_diagnostics().values())
    E2 = np.ascontiguousarray(E * (1.0 + 0.5 * np.random.default_rng(L).random((L, 1))))
    assert not _allocate(plan, E2, Kt, budget, D)["rows_decided"]
    plan.close()


@pytest.mark.parametrize("cells,L,J,want", [(4225, 23, 16, "rows"), (4225, 24, 16, "halves"), (4225, 15, 17, "rows"), (4225, 16, 17, "halves"),
                                           (16383, 23, 16, "rows"), (16384, 15, 16, "rows"), (16384, 16, 16, "halves"),
                                           (575, 63, 8, "rows"), (575, 64, 8, "tree"), (576, 59, 8, "rows"), (576, 60, 8, "tree"),
                                           (1536, 59, 8, "rows"), (1537, 23, 8, "band"), (1537, 24, 8, "tree"), (90, 64, 8, "tree")])
def test_the_lines_where_halves_and_the_tree_begin(cells, L, J, want):
    ratios, sizes, Kt, E, budget, D = _case(cells, L, J, False)
    plan = _plan(sizes, ratios, D, budget)
    route = _allocate(plan, E, Kt, budget, D)
    assert route["route"] == want and not route["rows_decided"], route
    plan.close()


@pytest.mark.parametrize("flags,want", [(0, "halves"), (2, "rows"), (4, "halves")])
def test_rows_beyond_lds_know_no_band(flags, want):
    ratios, sizes, Kt, E, budget, D = _case(9000, 40, 12, False)
    plan = _plan(sizes, ratios, D, budget, flags)
    assert _allocate(plan, E, Kt, budget, D)["route"] == want
    plan.close()


def test_members_of_a_run_apart_by_rounding_are_told_apart_from_the_left():
    """Small layers whose sizes all cost one unit, of errors a few units in the last place of the total apart."""
    rng = np.random.default_rng(3)
    L, cells, J = 80, 700, 24
    ratios = np.append(np.sort(rng.uniform(0.05, 0.95, size=J - 1)), 1.0)
    sizes = [int(x) for x in np.where(np.arange(L) % 2, 150, rng.integers(3000, 20000, size=L))]
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    budget = 8 * (cells - 1) * (int(0.3 * sum(sizes)) // (cells - 1))
    unit = budget // 8 // (cells - 1)
    assert unit >= 150
    n = np.array(sizes, dtype=np.float64)[:, None]
    E = rng.uniform(1.0, 9.0, size=(L, 1)) * (1.0 - Kt / n) ** 2
    for near, left in ((1e-3, False), (4e-15, True)):
        Ek = E.copy()
        Ek[1::2] = 1.0 + near * np.arange(J)[::-1]
        plan = _plan(sizes, ratios, cells - 1, budget)
        route = _allocate(plan, np.ascontiguousarray(Ek), Kt, budget, cells - 1)
        assert route == dict(route="tree", rows_decided=False, from_left=left, at_once=False), (near, route)
        plan.close()


@pytest.mark.parametrize("cells,L,J", [(600, 64, 16), (1200, 70, 33), (4097, 40, 16), (4225, 24, 5), (9000, 20, 20)])
@pytest.mark.parametrize("recorded", [False, True])
def test_ties_in_a_row_go_by_whole_rows_at_once(cells, L, J, recorded):
    """Behind eight allocations that whole rows had to decide, the next 31 do not ask the tree or the halves first, whatever
    their tables; then it is tried again.  Called one by one, and as replays of a recorded graph."""
    import torch
    ratios, sizes, Kt, E, budget, D = _case(cells, L, J, True)
    clear = np.ascontiguousarray(E * (1.0 + 0.5 * np.random.default_rng(L).random((L, 1))))
    want = {id(t): ko.allocate(t, Kt, budget, 8, D) for t in (E, clear)}
    plan = _plan(sizes, ratios, D, budget)
    table = torch.empty(L * J, dtype=torch.float64, device="cuda")
    table.copy_(torch.from_numpy(clear.reshape(-1)))
    out = plan.allocate(budget, table)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    if recorded:
        with torch.cuda.graph(graph):
            out = plan.allocate(budget, table)

    def call(t):
        table.copy_(torch.from_numpy(t.reshape(-1)))
        for v in out:
            v.fill_(-7)
        if recorded:
            graph.replay()
        else:
            plan.allocate(budget, table)
        torch.cuda.synchronize()
        st_ref, j_ref, K_ref, off_ref = want[id(t)]
        j, K, off, st = out
        assert int(st.item()) == st_ref == ko.OK
        assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref)
        assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
        torch.full((1 << 18,), 1.0, device="cuda").sum().item()
        r = plan.allocate_route()
        assert r["route"] == ("halves" if cells > 4224 else "tree") and not r["from_left"]
        return r["rows_decided"], r["at_once"]

    assert [call(E) for _ in range(7)] == [(True, False)] * 7
    assert call(clear) == (False, False)                                 # (not in a row)
    assert [call(E) for _ in range(8)] == [(True, False)] * 8
    assert [call((E, clear)[k % 3 == 1]) for k in range(31)] == [(True, True)] * 31
    assert call(E) == (True, False)                                      # tried again, and again by rows
    assert [call(E) for _ in range(31)] == [(True, True)] * 31
    assert [call(clear) for _ in range(3)] == [(False, False)] * 3
    assert [call(E) for _ in range(7)] == [(True, False)] * 7
    plan.close()


@pytest.mark.parametrize("cells,L,J", [(900, 66, 12), (4100, 30, 40), (4225, 24, 5), (9000, 20, 20), (20011, 62, 33)])
def test_replays_of_a_recorded_allocation(cells, L, J):
    """Clear tables, ties and tables with a NaN one after another through one recorded graph, by the tree and by halves: what a replay
    leaves (counters, rows that the chain has refilled, the word that says it decides) is cleared by the next, with the program's own
    work and synchronizations in between."""
    import torch
    ratios, sizes, Kt, tied, budget, D = _case(cells, L, J, True)
    tables = {"tied": tied}
    for k in range(3):
        tables["clear%d" % k] = np.ascontiguousarray(tied * (1.0 + 0.5 * np.random.default_rng(L + k).random((L, 1))))
    tables["bad"] = tables["clear0"].copy()
    tables["bad"][L // 2, J // 2] = np.nan
    want = {k: ko.allocate(t, Kt, budget, 8, D) for k, t in tables.items()}
    plan = _plan(sizes, ratios, D, budget)
    table = torch.from_numpy(tied.reshape(-1).copy()).cuda()
    plan.allocate(budget, table)                         # (an eager call that the chain has decided)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        j, K, off, st = plan.allocate(budget, table)
    for k in ("tied", "clear0", "tied", "tied", "clear1", "bad", "clear2", "bad", "tied", "clear0"):
        table.copy_(torch.from_numpy(tables[k].reshape(-1)))
        for v in (j, K, off, st):
            v.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        st_ref, j_ref, K_ref, off_ref = want[k]
        assert int(st.item()) == st_ref == (ko.ERR_NONFINITE if k == "bad" else ko.OK), k
        if k == "bad":
            assert not j.cpu().numpy().any() and not K.cpu().numpy().any() and not off.cpu().numpy().any()
        else:
            assert np.array_equal(j.cpu().numpy(), j_ref), k
            assert np.array_equal(K.cpu().numpy().astype(np.uint64), K_ref) and np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), k
        route = plan.allocate_route()
        assert route["route"] == ("halves" if cells > 4224 else "tree") and route["rows_decided"] == (k == "tied") and not route["at_once"], (k, route)
        torch.full((1 << 20,), 2.0, device="cuda").sum().item()
        if k == "clear1":                                # an eager call on the plan between two replays
            j2, K2, off2, st2 = plan.allocate(budget, torch.from_numpy(tables["tied"].reshape(-1).copy()).cuda())
            assert np.array_equal(j2.cpu().numpy(), want["tied"][1])
    plan.close()
