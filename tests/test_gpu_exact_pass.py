"""The exact last-digit pass: layers whose entries share prefixes, so that no bound on what is dropped is tight.  A wave scans a
pool entry, a quarter of its 4096 digits at a time and sixteen digits a lane; the layer's last workgroup takes sixteen entries
at a time."""
import numpy as np
import pytest

from oracle import kimad_oracle as ko
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu

DIGITS = {
    "all": np.arange(4096), "first": np.array([0]), "last": np.array([4095]), "lanes": np.array([1615, 1616, 1631, 1632]),
    "quarters": np.array([1023, 1024, 2047, 2048, 3071, 3072]), "ends": np.array([0, 4095]), "one": np.array([1500]),
    "lanes' ends": np.array([1008, 1023]), "quarter": np.arange(2048, 3072),
}
CERTIFIED = {"first", "last"}


def _plan(x, sizes, ratios, flags):
    import torch
    import paper_2312_08053_amd as kimad
    g = torch.from_numpy(x).cuda()
    return g, kimad.Plan(g, torch.zeros_like(g), sizes, ratios, D=1000, max_budget_bytes=4 * len(x), cfg_flags=flags)


@pytest.mark.parametrize("flags", [0, 1])                # single pass, classic profile
@pytest.mark.parametrize("n", [8193, 40000, 300_001])
def test_one_prefix(n, flags):
    """A layer's entries all share one prefix: nothing but the scan's sum is in its errors.  That adds up at most 4096 + n products,
    forty roundings deep, so it is within 40 x 2^-53 < 1e-14 of the sum in extended precision.  Equal entries at an end of the
    prefix need no scan: there the bounds meet, and the error is certified to 4e-6."""
    rng = np.random.default_rng(n)
    ratios = np.linspace(0.03, 0.97, 48)
    keys = [((0x3A5 + 37 * k) << 19 | (17 + k) << 12) + rng.choice(d, size=n) for k, d in enumerate(DIGITS.values())]
    x = np.concatenate(keys).astype(np.uint32)
    x |= rng.integers(0, 2, size=len(x)).astype(np.uint32) << 31
    sizes = [n] * len(DIGITS)
    _, plan = _plan(x.view(np.float32), sizes, ratios.tolist(), flags)
    E = plan.profile(budget_hint_bytes=n).cpu().numpy().reshape(len(sizes), -1)
    K = ko.grid_sizes(ratios, n)
    for i, (name, k) in enumerate(zip(DIGITS, keys)):
        below = np.concatenate([[0], np.cumsum(np.sort(k.astype(np.uint32).view(np.float32)).astype(np.longdouble) ** 2)])
        want = below[n - K].astype(np.float64)
        assert np.all(np.abs(E[i] - want) <= (4e-6 if name in CERTIFIED else 1e-14) * want), name
    d = plan.diagnostics()
    scanned = len(sizes) - len(CERTIFIED)
    assert d["pool_entries"] == scanned and d["recomputed"] == 48 * scanned, d
    plan.close()


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("sizes", [[8193], [9000] * 5 + [200_000], [8200 + 61 * i for i in range(150)]])
def test_many_prefixes(sizes, flags):
    """Forty magnitudes a layer, a target near each: more pool entries than a workgroup has waves.  At the parity tests' bar (what is not
    scanned is certified to 4e-6)."""
    rng = np.random.default_rng(len(sizes))
    x = np.concatenate([(2.0 ** (rng.integers(0, 40, size=n) / 4.0) * 1.0123 * 10.0 ** rng.uniform(-4, -1)).astype(np.float32) for n in sizes])
    ratios = np.linspace(0.0125, 0.9875, 40)
    _, plan = _plan(x, sizes, ratios.tolist(), flags)
    E = plan.profile(budget_hint_bytes=4 * len(x)).cpu().numpy()
    Kt = np.array([ko.grid_sizes(ratios, s) for s in sizes])
    at = np.concatenate([[0], np.cumsum(sizes)])
    E_ref = np.array([ko.topk_error_profile(x[a:b], k) for a, b, k in zip(at[:-1], at[1:], Kt)])
    gh.assert_table_close(E, E_ref, Kt, sizes)
    assert plan.diagnostics()["pool_entries"] > 20 * len(sizes)
    plan.close()
