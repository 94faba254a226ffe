"""Small layers beside tiled ones, on both sides of the number up to which they share a launch of the main stream (512): beyond it
their kernels run on the plan's side stream, between a fork and a join.  Table, payload and estimator against the oracle."""
import numpy as np
import pytest

from kimad_synth.gen import Workload
from oracle import kimad_oracle as ko
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


def _sizes(small, seed):
    rng = np.random.default_rng(seed)
    s = [int(x) for x in np.minimum(8192, 10 ** rng.uniform(0, 3.0, size=small)).astype(np.int64)]
    s[0], s[-1] = 8192, 1
    at = sorted(rng.choice(small, size=4, replace=False))
    for k, n in zip(at[::-1], (8193, 70000, 25001, 1024 * 33)):
        s.insert(int(k), n)
    return s


def _draw(sizes, rng):
    return np.concatenate([10.0 ** rng.uniform(-4, -1) * rng.standard_t(3, size=n) for n in sizes]).astype(np.float32)


def _check(plan, sizes, ratios, g, h, hd, budget, table=True):
    work = Workload(name="many", sizes=np.asarray(sizes, dtype=np.uint64), g=g, h=h, ratios=ratios, budget_bytes=budget, cost_units_D=1000)
    gL, hL = gh.oracle_layers(work)
    if table:
        E_ref, Kt = ko.profile(gL, hL, ratios)
        gh.assert_table_close(plan.err_table.cpu().numpy(), E_ref, Kt, sizes)
    gh.check_compress(work, plan, hd, plan.K.cpu().numpy(), plan.offsets.cpu().numpy(), plan.idx, plan.val)


@pytest.mark.parametrize("flags", [0, 1])               # single pass, classic profile
@pytest.mark.parametrize("small", [511, 512, 513, 700])
def test_a_step_with_many_small_layers(small, flags):
    import torch
    import paper_2312_08053_amd as kimad
    sizes, ratios = _sizes(small, small), np.logspace(-2, 0, 12)
    rng = np.random.default_rng(small + 1)
    d = sum(sizes)
    gd, hd = torch.empty(d, device="cuda"), torch.zeros(d, device="cuda")
    budget = int(0.2 * 4 * d)
    plan = kimad.Plan(gd, hd, sizes, ratios.tolist(), D=4000, max_budget_bytes=budget, cfg_flags=flags)
    for step in range(3):
        g, h = _draw(sizes, rng), hd.cpu().numpy()
        gd.copy_(torch.from_numpy(g))
        assert plan.step(budget).cpu().tolist() == [0, 0]
        _check(plan, sizes, ratios, g, h, hd, budget)
    # selection from scratch at other sizes
    g, h = _draw(sizes, rng), hd.cpu().numpy()
    gd.copy_(torch.from_numpy(g))
    K = np.array([int(rng.integers(0, n + 1)) for n in sizes])
    plan.K.copy_(torch.from_numpy(K))
    plan.offsets.copy_(torch.from_numpy(np.concatenate([[0], np.cumsum(K)])))
    assert int(plan.compress_ef()[2].item()) == 0
    _check(plan, sizes, ratios, g, h, hd, budget, table=False)
    plan.close()


@pytest.mark.parametrize("small", [512, 700])
def test_recorded_with_many_small_layers(small):
    """The fork and the join are part of the recording; every replay meets another gradient, with the program's own work between."""
    import torch
    import paper_2312_08053_amd as kimad
    sizes, ratios = _sizes(small, 3 * small), np.logspace(-2, 0, 12)
    rng = np.random.default_rng(small + 2)
    d = sum(sizes)
    gd, hd = torch.zeros(d, device="cuda"), torch.zeros(d, device="cuda")
    budget = int(0.2 * 4 * d)
    plan = kimad.Plan(gd, hd, sizes, ratios.tolist(), D=4000, max_budget_bytes=budget)
    gd.copy_(torch.from_numpy(_draw(sizes, rng)))
    plan.step(budget)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.step(budget)
    for _ in range(4):
        g, h = _draw(sizes, rng), hd.cpu().numpy()
        gd.copy_(torch.from_numpy(g))
        graph.replay()
        torch.cuda.synchronize()
        assert plan.status.cpu().tolist() == [0, 0]
        _check(plan, sizes, ratios, g, h, hd, budget)
        torch.full((1 << 18,), 2.0, device="cuda").add_(1.0)
