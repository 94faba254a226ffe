"""Selection and payload, bit for bit against the oracle, at the sizes where the kernels that look after a layer change
or end: layers served from g and h throughout (more is kept than a layer's candidate region holds), layers sorted or
selected whole in LDS."""
import numpy as np
import pytest

from kimad_synth.gen import Workload
from oracle import kimad_oracle as ko
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


def _layers(sizes, seed, ties):
    rng = np.random.default_rng(seed)
    g = [(rng.standard_t(3, size=n) * 10.0 ** rng.uniform(-4, 0)).astype(np.float32) for n in sizes]
    if ties:
        g = [np.round(x / np.abs(x).max() * 40).astype(np.float32) for x in g]     # few magnitudes: every threshold is tied
    h = [(0.3 * rng.standard_normal(n) * np.abs(x).mean()).astype(np.float32) if not ties else np.zeros(n, np.float32)
         for n, x in zip(sizes, g)]
    return np.concatenate(g), np.concatenate(h)


def _compress(sizes, K, seed, ties, shift, f16=False):
    import torch
    import paper_2312_08053_amd as kimad
    g, h = _layers(sizes, seed, ties)
    n = g.size
    gd, hd = (torch.empty(n + shift, dtype=torch.float32, device="cuda")[shift:] for _ in range(2))
    gd.copy_(torch.from_numpy(g)); hd.copy_(torch.from_numpy(h))
    off = np.concatenate([[0], np.cumsum(K)])
    plan = kimad.Plan(gd, hd, list(sizes), [1.0], capacity_pairs=int(off[-1]), value_format=1 if f16 else 0,
                      max_budget_bytes=8)
    idx, val, st = plan.compress_ef(torch.tensor(K).cuda(), torch.from_numpy(off).cuda())
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    work = Workload(name="sel", sizes=np.asarray(sizes, dtype=np.uint64), g=g, h=h, ratios=np.array([1.0]),
                    budget_bytes=8, cost_units_D=0)
    gh.check_compress(work, plan, hd, K, off, idx, val)
    return plan


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_layers_served_from_g_and_h(shift, ties):
    sizes = [8193, 9215, 9216, 9217, 65536 + 1021, 8200, 12345, 30001]
    K = [8193, 9214, 4700, 8000, 65000, 1, 12344, 30001]
    plan = _compress(sizes, K, 5, ties, shift)
    assert 4 in [s["mode"] for s in plan.layer_states()]


@pytest.mark.parametrize("ties", [False, True])
def test_small_layers_of_every_shape(ties):
    sizes = [1, 2, 3, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 2049, 4095, 4097, 8191, 8192, 8192, 8192, 700]
    K = [1, 1, 3, 5, 64, 64, 1, 100, 513, 1022, 1, 600, 2048, 4095, 17, 8191, 8192, 4096, 1, 0]
    _compress(sizes, K, 6, ties, 1)


@pytest.mark.parametrize("largest", [1048576 + 77, 2900000, 3145728])
@pytest.mark.parametrize("share", [0.0, 0.001, 0.06, 0.124, 0.13, 0.7, 1.0])
def test_selection_from_scratch_over_several_rounds(share, largest):
    """One size per layer, from histogram passes (the smaller sets) and from the single pass (the largest: 3287 chunks):
    the first call predicts from a sample, the later ones from the histogram of the call before; a gradient scaled by 64
    in between makes every prediction miss."""
    import torch
    import paper_2312_08053_amd as kimad
    sizes = [9000, 200001, 5000, largest, 8193]
    K = [min(n, int(np.ceil(share * n))) for n in sizes]
    off = np.concatenate([[0], np.cumsum(K)])
    g, h = _layers(sizes, 7, False)
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    plan = kimad.Plan(gd, hd, sizes, [1.0], capacity_pairs=max(1, int(off[-1])), max_budget_bytes=8)
    Kd, offd = torch.tensor(K).cuda(), torch.from_numpy(off).cuda()
    for scale in (1.0, 1.1, 64.0, 1.0):
        g1 = (g * np.float32(scale)).astype(np.float32)
        gd.copy_(torch.from_numpy(g1))
        h0 = hd.cpu().numpy()
        idx, val, st = plan.compress_ef(Kd, offd)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        work = Workload(name="scratch", sizes=np.asarray(sizes, dtype=np.uint64), g=g1, h=h0, ratios=np.array([1.0]),
                        budget_bytes=8, cost_units_D=0)
        gh.check_compress(work, plan, hd, K, off, idx, val)


@pytest.mark.parametrize("zeros", [0.0, 0.015, 0.3])
@pytest.mark.parametrize("n", [8193, 70001, 400003])
def test_profile_on_a_grid_up_to_nearly_all_entries(n, zeros):
    """The paper's grid needs digit-2 tables over more bins than one run of them covers, and more spilled than the
    budget asks for; with exact zeros in the layer, a ratio's boundary lies among them."""
    import torch
    import paper_2312_08053_amd as kimad
    from kimad_synth.gen import paper_grid
    rng = np.random.default_rng(n)
    sizes, ratios = [n, n, 12000], paper_grid()
    gd = torch.empty(sum(sizes), dtype=torch.float32, device="cuda")
    hd = torch.zeros_like(gd)
    plan = kimad.Plan(gd, hd, sizes, ratios.tolist(), D=1000, max_budget_bytes=4 * sum(sizes))
    Kt = plan.grid_sizes()
    starts = np.concatenate([[0], np.cumsum(sizes)])
    for _ in range(3):
        g = rng.standard_t(3, size=sum(sizes)).astype(np.float32)
        g[rng.random(g.size) < zeros] = 0.0
        gd.copy_(torch.from_numpy(g))
        E = plan.profile(budget_hint_bytes=int(0.05 * 4 * sum(sizes))).cpu().numpy().reshape(len(sizes), -1)
        gL = [g[a:b] for a, b in zip(starts[:-1], starts[1:])]
        E_ref, _ = ko.profile(gL, [np.zeros_like(x) for x in gL], ratios)
        gh.assert_table_close(E, E_ref, Kt, sizes)
    if n == 400003:
        assert plan.diagnostics()["redo_layers"] <= 1       # (the layer of 12000 entries may be recounted)


@pytest.mark.parametrize("D", [30, 60, 1000])
def test_layers_that_pay_for_a_whole_cost_unit_are_served_from_the_candidates(D):
    """Layers far below the budget's cut still get what one cost unit holds, more than a four-hundredth of a layer where
    units are coarse: the pass spills that much of them, so nothing is read a second time."""
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(3)
    sizes = [200000 + 13 * i for i in range(12)]
    ratios = np.logspace(-4, 0, 48)
    d = sum(sizes)
    budget = int(0.02 * 4 * d)
    gd = torch.empty(d, dtype=torch.float32, device="cuda")
    hd = torch.zeros_like(gd)
    plan = kimad.Plan(gd, hd, sizes, ratios.tolist(), D=D, max_budget_bytes=budget)
    scales = np.repeat(10.0 ** np.linspace(-5, -2, len(sizes)), sizes)
    for _ in range(3):
        g = (rng.standard_t(3, size=d) * scales).astype(np.float32)
        gd.copy_(torch.from_numpy(g))
        hd.zero_()
        assert plan.step(budget).cpu().tolist() == [0, 0]
        K = plan.K.cpu().numpy()
        assert all(s["mode"] == 3 for s in plan.layer_states()), (K, plan.layer_states())
        work = Workload(name="units", sizes=np.asarray(sizes, dtype=np.uint64), g=g, h=np.zeros_like(g), ratios=ratios,
                        budget_bytes=budget, cost_units_D=D)
        gh.check_compress(work, plan, hd, K.tolist(), np.concatenate([[0], np.cumsum(K)]), plan.idx, plan.val)


@pytest.mark.parametrize("L", [100, 103, 154, 420])
def test_recount_in_groups_of_tiles(L):
    """Layers of a few tiles each, so that a group of tiles ends inside a layer, spans several, or is one tile: below and
    above the tiles per compute unit from which on groups form."""
    import torch
    import paper_2312_08053_amd as kimad
    from paper_2312_08053_amd import binding
    rng = np.random.default_rng(L)
    sizes = [8193 + 2048 * int(rng.integers(0, 2)) + i % 7 for i in range(L)]
    ratios = np.logspace(-2, 0, 12)
    g = (rng.standard_t(3, size=sum(sizes)) * 1e-3).astype(np.float32)
    g[rng.random(g.size) < 0.02] = 0.0
    gd = torch.from_numpy(g).cuda()
    plan = kimad.Plan(gd, torch.zeros_like(gd), sizes, ratios.tolist(), D=1000, max_budget_bytes=8 * sum(sizes),
                      cfg_flags=binding.KIMAD_CFG_CLASSIC_PROFILE)
    E = plan.profile().cpu().numpy().reshape(L, -1)
    starts = np.concatenate([[0], np.cumsum(sizes)])
    gL = [g[a:b] for a, b in zip(starts[:-1], starts[1:])]
    E_ref, _ = ko.profile(gL, [np.zeros_like(x) for x in gL], ratios)
    gh.assert_table_close(E, E_ref, plan.grid_sizes(), sizes)


@pytest.mark.parametrize("share", [0.02, 0.3, 0.9])
@pytest.mark.parametrize("sizes", [[8193, 12289, 40003, 9216], [17_000_001, 8193, 300_001]])
def test_thresholds_among_equal_magnitudes(sizes, share):
    """More is kept than lies above a magnitude that many entries share: zeros in the first layer; in the others two
    magnitudes of one prefix bin, in runs of one chunk, of one quad and of one entry (the larger set has more tiles than
    the pass has workgroups, and a layer's neighbours have a run of the same digit)."""
    import torch
    import paper_2312_08053_amd as kimad
    rng = np.random.default_rng(11)
    g = []
    for i, n in enumerate(sizes):
        near = np.array([1.0, np.float32(1.0) + np.float32(2.0 ** -22)], dtype=np.float32)
        x = np.zeros(n, np.float32) if i == 0 else near[(np.arange(n) // [1024, 4, 1][i % 3]) % 2]
        some = rng.choice(n, n // 200, replace=False)
        x[some] = rng.standard_normal(some.size) * 10
        g.append(x)
    g = np.concatenate(g)
    h = np.zeros_like(g)
    K = [int(share * n) for n in sizes]
    off = np.concatenate([[0], np.cumsum(K)])
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    plan = kimad.Plan(gd, hd, sizes, [1.0], capacity_pairs=int(off[-1]), max_budget_bytes=8)
    idx, val, st = plan.compress_ef(torch.tensor(K).cuda(), torch.from_numpy(off).cuda())
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    work = Workload(name="ties", sizes=np.asarray(sizes, dtype=np.uint64), g=g, h=h, ratios=np.array([1.0]),
                    budget_bytes=8, cost_units_D=0)
    gh.check_compress(work, plan, hd, K, off, idx, val)
