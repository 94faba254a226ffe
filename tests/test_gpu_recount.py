"""Layers whose prediction misses are recounted, and scanned by the workgroup that adds the last of their tiles; a layer of many
parts is summed by whole workgroups, one of few by a wave a block.  Short layers, several to a workgroup, beside one of more
than sixteen parts: the first round predicts from a sample, the second is 64 times the first, so that every layer is recounted,
the third comes back.  The table against the oracle at the parity tests' bar, and against a plan that samples, bit for bit."""
import numpy as np
import pytest

from kimad_synth.gen import Workload
from oracle import kimad_oracle as ko
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("short,lo,hi,long", [(1, 8193, 8194, 0), (40, 8193, 9500, 400_001), (70, 8200, 30000, 0)])
@pytest.mark.parametrize("J", [5, 64])
def test_recounted_layers(short, lo, hi, long, J):
    import torch
    from paper_2312_08053_amd.binding import KIMAD_CFG_SAMPLE_ALWAYS
    rng = np.random.default_rng(short + J)
    sizes = [int(x) for x in rng.integers(lo, hi, size=short)] + ([long] if long else [])
    n = int(sum(sizes))
    base = (rng.standard_t(3, size=n) * np.repeat(10.0 ** rng.uniform(-4, -1, size=len(sizes)), sizes)).astype(np.float32)
    ratios = np.geomspace(1e-3, 1.0, J)
    w = Workload(name="recount", sizes=np.array(sizes, dtype=np.uint64), g=base, h=np.zeros(n, np.float32), ratios=ratios,
                 budget_bytes=int(0.04 * n), cost_units_D=500)
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes])
    g, h = gh.to_device(w)
    plan, ref = gh.make_plan(w, g, h), gh.make_plan(w, g, h, cfg_flags=KIMAD_CFG_SAMPLE_ALWAYS)
    redone = []
    for factor in (1.0, 64.0, 1.0):
        x = base * np.float32(factor)
        g.copy_(torch.from_numpy(x))
        E = plan.profile(budget_hint_bytes=w.budget_bytes).cpu().numpy().copy()
        other = ref.profile(budget_hint_bytes=w.budget_bytes).cpu().numpy()
        assert np.array_equal(E, other)
        redone.append(plan.diagnostics()["redo_layers"])
        start = np.concatenate([[0], np.cumsum(sizes)])
        E_ref = np.array([ko.topk_error_profile(x[a:b], Kt[i]) for i, (a, b) in enumerate(zip(start[:-1], start[1:]))])
        gh.assert_table_close(E, E_ref, Kt, sizes)
    assert redone[1] == len(sizes)
    plan.close()
    ref.close()


def test_more_layers_than_a_workgroup_reports_at_once():
    """20 thousand layers of one or two chunks more than the smallest tiled one: every workgroup of the recount counts more runs
    than it keeps, and reports and scans in between."""
    import torch
    import paper_2312_08053_amd as kimad
    from paper_2312_08053_amd.binding import KIMAD_CFG_SAMPLE_ALWAYS
    sizes = [8193 + 7 * (i % 3) for i in range(20000)]
    n, J = sum(sizes), 3
    ratios = [0.001, 0.02, 0.3]
    gen = torch.Generator(device="cuda").manual_seed(3)
    base = torch.randn(n, generator=gen, device="cuda")
    g, h = base.clone(), torch.zeros(n, device="cuda")
    plans = [kimad.Plan(g, h, sizes, ratios, D=1000, max_budget_bytes=n // 10, cfg_flags=f, capacity_pairs=1) for f in (0, KIMAD_CFG_SAMPLE_ALWAYS)]
    start = np.concatenate([[0], np.cumsum(sizes)])
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes])
    which = [0, 1, 2, 9999, 19998, 19999]
    for factor in (1.0, 64.0):
        torch.mul(base, factor, out=g)
        tables = [p.profile(budget_hint_bytes=n // 10).cpu().numpy().reshape(len(sizes), J) for p in plans]
        print("profiled", factor, flush=True)
        assert np.array_equal(tables[0], tables[1])
        x = {i: g[start[i]:start[i + 1]].cpu().numpy() for i in which}
        E_ref = np.array([ko.topk_error_profile(x[i], Kt[i]) for i in which])
        gh.assert_table_close(tables[0][which], E_ref, Kt[which], [sizes[i] for i in which])
    assert plans[0].diagnostics()["redo_layers"] == len(sizes)
    for p in plans:
        p.close()
