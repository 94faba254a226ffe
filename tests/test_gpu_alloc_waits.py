"""The allocation's workgroups wait for one another's cells, and the waits are bounded: with the first workgroup withheld and a
short bound, set from the host, every kernel ends by itself, the call reports an internal error with zero-filled outputs, and
the plan's next allocation is the oracle's.  The number past the last one, which is given out instead, owns no cells."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko
from tests.test_gpu_alloc_chain import _case, _plan

pytestmark = pytest.mark.gpu
INTERNAL = -9


def _withheld(plan, table, budget, polls):
    import torch
    import paper_2312_08053_amd.binding as b
    j, K = torch.full_like(plan.j, 7), torch.full_like(plan.K, 7)
    off, st = torch.full_like(plan.offsets, 7), torch.zeros(1, dtype=torch.int32, device="cuda")
    waits = torch.zeros(1, dtype=torch.int32, device="cuda")
    b.kimad_selftest_allocate_withheld(plan.handle, table, budget, j, K, off, st, polls, waits)
    torch.cuda.synchronize()
    assert int(st.item()) == INTERNAL
    assert not j.cpu().numpy().any() and not K.cpu().numpy().any() and not off.cpu().numpy().any()
    return int(waits.item())


# one workgroup and many of each width, and the single waves of rows beyond LDS
@pytest.mark.parametrize("cells,L", [(40, 3), (65, 3), (700, 9), (1024, 130), (1024, 193), (2000, 20), (4224, 7), (4300, 3), (20011, 12)])
@pytest.mark.parametrize("J", [5, 20, 40])
def test_a_workgroup_that_never_comes_ends_in_an_error(cells, L, J):
    import torch
    ratios, sizes, Kt, E = _case(cells, J, L, 100 * cells + J)
    budget = 8 * (cells - 1)
    plan = _plan(sizes, ratios, budget)
    table = torch.from_numpy(E.reshape(-1)).cuda()
    # a wave gives up once, however many layers it still has to bring cells for
    cap = min(cells - 1, int(Kt[:, -1].sum()))
    per, loaders = (64, 4) if cap < 1024 and L > 128 else (128, 4) if cap < 1024 else (128, 6) if cap < 2048 else (64, 10) if cap < 4224 else (64, 1)
    waits = _withheld(plan, table, budget, 16)
    assert 0 < waits <= (cap // per + 1) * loaders + 1
    st_ref, j_ref, K_ref, off_ref = ko.allocate(E, Kt, budget, 8, 0)
    j, K, off, st = plan.allocate(budget, table)
    assert int(st.item()) == st_ref == ko.OK
    assert np.array_equal(j.cpu().numpy(), j_ref) and np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    plan.close()
