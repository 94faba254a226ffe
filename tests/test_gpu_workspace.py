"""A workspace without room for the rows that only make the exact cost axis faster: accepted, never written past its end, and the
same results by a launch per layer."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko
from tests.test_gpu_alloc_chain import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,L,J", [(4700, 3, 7), (20011, 12, 20), (60000, 40, 33)])
def test_a_workspace_without_all_rows_serves_the_plan(cells, L, J):
    import torch
    import paper_2312_08053_amd.binding as b
    ratios, sizes, Kt, E = _case(cells, J, L, 7 * cells + J)
    assert sum(sizes) >= cells
    budget = 8 * (cells - 1)
    total = b.kimad_workspace_bytes(sizes, J, D=0, max_budget_bytes=budget)
    spared = 8 * (L + 1) * (cells - 4608)
    assert 8 * (L + 1) * (cells + 127) <= 256 << 20
    n = int(sum(sizes))
    g, h = torch.randn(n, device="cuda"), torch.zeros(n, device="cuda")
    starts = np.concatenate([[0], np.cumsum(sizes)])[:-1] * 4
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
    table = torch.from_numpy(E.reshape(-1)).cuda()
    for size in (total, total - spared // 2, total - spared):
        ws = torch.full((total + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        off = -ws.data_ptr() % 256
        plan = b.kimad_plan_create([g.data_ptr() + int(s) for s in starts], [h.data_ptr() + int(s) for s in starts], sizes, ratios,
                                   ws.data_ptr() + off, size, D=0, max_budget_bytes=budget)
        try:
            j, st = torch.zeros(L, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
            K, o = torch.zeros(L, dtype=torch.int64, device="cuda"), torch.zeros(L + 1, dtype=torch.int64, device="cuda")
            err = torch.empty(L * J, dtype=torch.float64, device="cuda")
            b.kimad_profile(plan, err, budget)
            b.kimad_allocate(plan, table, budget, j, K, o, st)
            assert int(st.item()) == st_ref == ko.OK
            assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(o.cpu().numpy().astype(np.uint64), off_ref)
            assert bool((ws[off + size:] == 0xA5).all())
        finally:
            torch.cuda.synchronize()
            b.kimad_plan_destroy(plan)


def test_a_workspace_that_is_too_small_is_refused():
    import torch
    import paper_2312_08053_amd.binding as b
    n = [5000, 20000, 9000]
    g, h = torch.zeros(sum(n), device="cuda"), torch.zeros(sum(n), device="cuda")
    ptr = [4 * s for s in (0, 5000, 25000)]
    # (in turn: rows beyond LDS whose speed rows are left out and then some, rows within LDS, discretised costs)
    for D, budget, spared in ((0, 8 * 20000, 8 * 4 * (20001 + 128 - 4608)), (0, 8 * 3000, 0), (1000, 8 * 20000, 0)):
        total = b.kimad_workspace_bytes(n, 16, D=D, max_budget_bytes=budget)
        ws = torch.empty(total + 256, dtype=torch.uint8, device="cuda")
        at = ws.data_ptr() + -ws.data_ptr() % 256
        with pytest.raises(b.KimadError) as e:
            b.kimad_plan_create([g.data_ptr() + p for p in ptr], [h.data_ptr() + p for p in ptr], n, np.logspace(-2, 0, 16).tolist(),
                                at, total - spared - 256, D=D, max_budget_bytes=budget)
        assert e.value.code == -2
