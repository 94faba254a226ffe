"""The recurrence by workgroups that keep their own cost cells, and by waves on rows too long for LDS, at the edges of their
shapes: last cells of a workgroup, of the LDS rows and of the stored ones, candidate counts around the sixteens that a
register set holds, one layer, more layers than a record ring.  The oracle's dynamic programme, bit for bit."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko

pytestmark = pytest.mark.gpu

FULL = 2


def _case(cells, J, L, seed, ties=None):
    rng = np.random.default_rng(seed)
    ratios = np.sort(rng.uniform(0.0, 1.0, size=J)) ** 3 + np.linspace(1e-6, 1e-3, J)
    ratios = np.minimum(ratios / ratios[-1], 1.0)
    lo = max(2, cells // (4 * L))
    sizes = [int(x) for x in rng.integers(lo, 8 * lo + 40, size=L)]
    Kt = np.array([ko.grid_sizes(ratios, n) for n in sizes])
    E = np.sort(rng.random((L, J)) * 10.0 ** rng.uniform(-6, 6, size=(L, 1)), axis=1)[:, ::-1].copy()
    if seed % 3 == 0 if ties is None else ties:
        E = np.round(E, 1)                       # ties between totals
    return ratios, sizes, Kt, E


def _plan(sizes, ratios, budget):
    import torch
    import paper_2312_08053_amd as kimad
    n = int(sum(sizes))
    z = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2)]
    return kimad.Plan(z[0], z[1], list(sizes), list(ratios), D=0, max_budget_bytes=budget, cfg_flags=FULL, capacity_pairs=1)


@pytest.mark.parametrize("cells", [2, 63, 64, 65, 129, 1024, 1025, 2048, 2049, 4224, 4225, 4289, 20011])
@pytest.mark.parametrize("J", [1, 5, 16, 17, 33, 64])
def test_edges_of_the_rows(cells, J):
    import torch
    for L in (1, 2, 3, 4, 5, 13, 130):
        if L >= cells or (L == 130 and cells not in (1024, 1025)):        # (many layers of short rows: narrower workgroups)
            continue
        ratios, sizes, Kt, E = _case(cells, J, L, 1000 * cells + 10 * J + L)
        budget = 8 * (cells - 1)
        st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
        plan = _plan(sizes, ratios, budget)
        for _ in range(2):                       # the rows of the call before are in the workspace
            j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
            assert int(st.item()) == st_ref, (cells, J, L)
            if st_ref == ko.OK:
                assert np.array_equal(j.cpu().numpy(), j_ref), (cells, J, L)
                assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), (cells, J, L)
        plan.close()


@pytest.mark.parametrize("cells,L,J", [(11263, 6, 16), (11264, 6, 16), (11329, 6, 5), (14335, 6, 17), (14336, 6, 17), (23551, 30, 6), (23552, 30, 6), (24064, 31, 6),
                                         (23551, 15, 40), (23552, 15, 40), (24577, 16, 40), (90111, 17, 20), (90112, 17, 20), (90177, 17, 6)])
def test_one_wave_a_workgroup_and_two(cells, L, J):
    """Around the lines from which a workgroup of rows beyond LDS has two waves, the last workgroup full, of one wave and nearly empty."""
    import torch
    ratios, sizes, Kt, E = _case(cells, J, L, cells + L)
    budget = 8 * (cells - 1)
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
    assert st_ref == ko.OK
    plan = _plan(sizes, ratios, budget)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == st_ref
    assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()


@pytest.mark.parametrize("cells", [200, 256, 257, 1000, 1030, 2049])
@pytest.mark.parametrize("L", [23, 24, 25, 28, 29, 61])
def test_pieces_that_the_walk_goes_through(cells, L):
    """The last 24 layers are followed back singly, the ones before in fours, the last of those shorter."""
    import torch
    ratios, sizes, Kt, E = _case(cells, 21, L, 3 * cells + L)          # (seeds that are multiples of 3: ties)
    budget = 8 * (cells - 1)
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
    plan = _plan(sizes, ratios, budget)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == st_ref
    if st_ref == ko.OK:
        assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("L,cells", [(L, c) for L in (25, 28, 29, 61) for c in (257, 1000, 1030, 2049)] +
                         [(191, 1000), (192, 1000), (193, 300), (193, 1000), (193, 1024), (193, 1025), (220, 2049)])
def test_ties_within_pieces(L, cells, ties):
    """Layers in pieces of four, with equal totals and without, in each of the kernels of rows that fit LDS (four waves a
    workgroup beyond 192 layers of up to 1024 cells, and beyond 2048 cells)."""
    import torch
    ratios, sizes, Kt, E = _case(cells, 21, L, 5 * cells + L, ties)
    budget = 8 * (cells - 1)
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
    assert st_ref == ko.OK
    plan = _plan(sizes, ratios, budget)
    j, K, off, st = plan.allocate(budget, torch.from_numpy(E.reshape(-1)).cuda())
    assert int(st.item()) == st_ref
    assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()


@pytest.mark.parametrize("cells", [700, 9000])
def test_non_finite_errors_end_the_call(cells):
    import torch
    for bad in (np.inf, -np.inf, np.nan):
        ratios, sizes, Kt, E = _case(cells, 20, 7, 3)
        E[3, 4] = bad
        plan = _plan(sizes, ratios, 8 * (cells - 1))
        j, K, off, st = plan.allocate(8 * (cells - 1), torch.from_numpy(E.reshape(-1)).cuda())
        st_ref = ko.allocate(E, Kt, 8 * (cells - 1), 8, 0)[0]
        assert int(st.item()) == st_ref != ko.OK and not K.cpu().numpy().any()
        plan.close()


@pytest.mark.parametrize("cells", [1000, 9000])
def test_recorded_into_a_graph(cells):
    """Every replay clears what the one before has left, with other tables and the program's own work in between."""
    import torch
    ratios, sizes, Kt, E = _case(cells, 24, 11, 8)
    budget = 8 * (cells - 1)
    plan = _plan(sizes, ratios, budget)
    table = torch.from_numpy(E.reshape(-1)).cuda()
    plan.allocate(budget, table)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        j, K, off, st = plan.allocate(budget, table)
    for k in range(4):
        Ek = E * (1.0 + 0.3 * np.sin(np.arange(E.size).reshape(E.shape) * (k + 1)))
        table.copy_(torch.from_numpy(Ek.reshape(-1)))
        graph.replay()
        torch.cuda.synchronize()
        st_ref, j_ref, K_ref, off_ref = ko.allocate(Ek, Kt, budget, 8, 0)
        assert int(st.item()) == st_ref == ko.OK
        assert np.array_equal(j.cpu().numpy(), j_ref), k
        assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref), k
        torch.full((1 << 20,), float(k), device="cuda").sum().item()
