"""The recount deals out the tiles of the recounted layers alone while a set has at most 768 tiled layers, and all tiles beyond:
a few layers among 1, 63, 768 and 769, the first and the last among them, miss their prediction, in lists that end inside a
wave and on its edge.  The table against a plan that samples in every round, bit for bit, and these layers' rows against the
oracle at the parity tests' bar."""
import numpy as np
import pytest

from kimad_synth.gen import Workload
from oracle import kimad_oracle as ko
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,moved", [(1, [0]), (63, [0, 31, 62]), (70, list(range(64))), (768, [0, 63, 64, 500, 767]), (769, [0, 512, 768])])
def test_a_few_recounted_among_many(layers, moved):
    import torch
    from paper_2312_08053_amd.binding import KIMAD_CFG_SAMPLE_ALWAYS
    rng = np.random.default_rng(layers)
    sizes = rng.integers(8193, 12000, size=layers)
    sizes[moved[-1]] = 70_001
    n = int(sizes.sum())
    base = (rng.standard_t(3, size=n) * 0.01).astype(np.float32)
    ratios = np.geomspace(1e-3, 1.0, 5)
    w = Workload(name="listed", sizes=sizes.astype(np.uint64), g=base, h=np.zeros(n, np.float32), ratios=ratios,
                 budget_bytes=int(0.04 * n), cost_units_D=500)
    g, h = gh.to_device(w)
    plan, ref = gh.make_plan(w, g, h), gh.make_plan(w, g, h, cfg_flags=KIMAD_CFG_SAMPLE_ALWAYS)
    plan.profile(budget_hint_bytes=w.budget_bytes)
    start = np.concatenate([[0], np.cumsum(sizes)])
    x = base.copy()
    for i in moved:
        x[start[i]:start[i + 1]] *= np.float32(64.0)
    g.copy_(torch.from_numpy(x))
    E = plan.profile(budget_hint_bytes=w.budget_bytes).cpu().numpy().copy()
    other = ref.profile(budget_hint_bytes=w.budget_bytes).cpu().numpy()
    assert np.array_equal(E, other)
    assert plan.diagnostics()["redo_layers"] >= len(moved)
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes[moved]])
    E_ref = np.array([ko.topk_error_profile(x[start[i]:start[i + 1]], Kt[r]) for r, i in enumerate(moved)])
    gh.assert_table_close(E.reshape(layers, 5)[moved], E_ref, Kt, sizes[moved])
    plan.close()
    ref.close()
