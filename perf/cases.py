"""The work that a user of this library has it do, as cases that can be timed and compared.

One round of a worker (profile, allocation, compression: ``Plan.step``) over the gradient sets of
``kimad_synth`` and over generic ragged ones; the same round with the allocation beside the next one; the round of
the method without the layer-wise allocation (one ratio for all layers, selection from scratch); and the server's
side of a round.  Sizes, value distributions, grids, budgets and cost axes are those of ``kimad_synth`` and
``bench.py`` or lie around them.

A trainer that lets the next backward pass write while this round's gradient is compressed keeps two gradient
buffers and one estimator: a state holds two such buffers, each with its plan, and passes alternate between them.
Every pass therefore meets a gradient that the estimator has not absorbed yet, as in training, and the estimator
carries over from pass to pass.  ``prepare`` runs one round on each plan: a round in the middle of training, not the
very first one, is what is timed.
"""
from __future__ import annotations

import math
import random

import torch

import kimad_synth as ks
import paper_2312_08053_amd as kimad
from kimad_synth.gen import paper_grid
from paper_2312_08053_amd import binding
from paper_2312_08053_amd.blocks import merge_small

# value distribution and range of the per-layer scales (powers of ten) of the named sets
RECIPES = {
    "normal": (-4.0, -1.0),
    "t3": (-5.0, -2.0),
    "laplace": (-6.0, -2.0),
    "t2.5": (-5.0, -2.0),
}


def _case(name, op, arch, **kw):
    c = dict(name=name, op=op, arch=arch, a=0, b=0, c=0, dist="t3", h_factor=0.0, grid="log64", budget=0.01, D=1000,
             f16=False, dense=False, block_min=0, h_shift=0, workers=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest set there is: a perceptron of six tensors, the exact cost axis; launches and latency count
        _case("mlp_step", "step", "mlp", dist="normal", grid="log16", budget=0.10, D=0),
        # the paper's own experiment: ResNet-18 with ten classes, the grid {0.01 + 0.02 k}, D = 1000
        _case("resnet18_paper_step", "step", "resnet18", a=10, grid="paper", budget=0.05),
        # ResNet-18 with the exact cost axis (58 thousand cells a row) and an estimator that is not zero
        _case("resnet18_exact_step", "step", "resnet18", a=1000, h_factor=0.5, grid="log32", D=0),
        # ResNet-50: 161 tensors, most of them small
        _case("resnet50_step", "step", "resnet50", a=1000, dist="laplace", grid="log32"),
        # ResNet-50 over a wide link with the dense fallback: many layers are sent whole
        _case("resnet50_wide_link_step", "step", "resnet50", a=1000, dist="laplace", grid="log32", budget=0.40, dense=True),
        # the headline workload of bench.py
        _case("gpt2_step", "step", "gpt2", a=12, b=768, c=50257, dist="t2.5"),
        # the same with rows of 4097 cells, half-precision values and a running estimator
        _case("gpt2_step_D4096_f16", "step", "gpt2", a=12, b=768, c=50257, dist="t2.5", h_factor=0.5, D=4096, f16=True),
        # the same with the allocation beside the next round (sizes one round old)
        _case("gpt2_overlapped_round", "overlap", "gpt2", a=12, b=768, c=50257, dist="t2.5"),
        # one ratio for all layers, sizes off the grid: selection from scratch
        _case("gpt2_uniform_ratio", "uniform", "gpt2", a=12, b=768, c=50257, dist="t2.5"),
        # the largest set
        _case("llama_step", "step", "llama", a=24, b=2048, c=32000),
        # the server's side: a small model with many workers, and the headline model with four
        _case("resnet18_server_16", "server", "resnet18", a=1000, workers=16),
        _case("gpt2_server_4", "server", "gpt2", a=12, b=768, c=50257, workers=4),
    ]


def _draw_arch(rng, most):
    """One model of the named kinds, or a ragged list of tensors, of at most `most` elements."""
    while True:
        kind = rng.choice(["ragged", "ragged", "resnet18", "resnet50", "gpt2", "llama"])
        if kind == "ragged":
            # a: seed of the sizes, b: tensors, c: elements in all
            arch = dict(arch=kind, a=rng.randrange(1, 1 << 30), b=int(round(math.exp(rng.uniform(math.log(3), math.log(400))))),
                        c=int(math.exp(rng.uniform(math.log(1.5e5), math.log(min(most, 1e9))))), dist=rng.choice(sorted(RECIPES)))
        elif kind == "resnet18":
            arch = dict(arch=kind, a=rng.randrange(2, 5000), dist="t3")
        elif kind == "resnet50":
            arch = dict(arch=kind, a=rng.randrange(2, 5000), dist="laplace")
        elif kind == "gpt2":
            arch = dict(arch=kind, a=rng.randrange(1, 25), b=64 * rng.randrange(2, 17), c=rng.randrange(500, 60000), dist="t2.5")
        else:
            arch = dict(arch=kind, a=rng.randrange(1, 25), b=128 * rng.randrange(2, 17), c=rng.randrange(1000, 40000), dist="t3")
        if sum(_sizes(_case("", "step", **arch))) <= most:
            return arch


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "overlap", "uniform", "server"])
    if op == "server":
        workers = rng.choice([1, 2, 3, 4, 8, 16])
        return {k: v for k, v in _case("", op, **_draw_arch(rng, 2e9 / (workers + 2)), workers=workers,
                                       budget=rng.choice([0.001, 0.01, 0.05])).items() if k != "name"}
    arch = _draw_arch(rng, 3.5e8 if op == "uniform" else 1.25e9)
    grid = rng.choice(["log16", "log32", "log64", "paper"])
    # (the paper's grid cannot spend less than a hundredth of the entries)
    budget = rng.choice([0.03, 0.05, 0.1, 0.2] if grid == "paper" else [0.001, 0.003, 0.01, 0.03, 0.1, 0.4])
    c = _case("", op, **arch, grid=grid, budget=budget, h_factor=rng.choice([0.0, 0.5]), D=rng.choice([500, 1000, 1000, 4096]),
              f16=rng.random() < 0.25, dense=rng.random() < 0.25, block_min=rng.choice([0, 0, 0, 8193]),
              h_shift=rng.choice([0, 0, 0, 1]))
    sizes = _sizes(c)
    if rng.random() < 0.3 and len(sizes) <= 170 and budget * 4 * sum(sizes) / _pair(c) <= 1.3e5:
        c["D"] = 0
    if sum(sizes) > 4e8 and budget > 0.05:
        c["budget"] = 0.05      # (wide links cost several passes over g and h: not over the largest models as well)
    # a budget that the cheapest sizes do not fit is no round: the next larger one is taken
    while not _feasible(c):
        c["budget"] *= 2
    c.pop("name")
    return c


def _feasible(case):
    pairs = _budget(case) // _pair(case)
    unit = 1 if case["D"] == 0 or pairs <= case["D"] else -(-pairs // case["D"])
    r0 = _ratios(case)[0]
    return sum(-(-max(1, math.ceil(r0 * n)) // unit) for n in _sizes(case)) <= pairs // unit


def _pair(case):
    return 6 if case["f16"] else 8


def _sizes(case):
    k, a, b, c = case["arch"], case["a"], case["b"], case["c"]
    if k == "ragged":
        # sizes spread over their logarithm, scaled to the total, odd ones among them
        r = random.Random(a)
        w = [math.exp(r.uniform(0.0, 9.0)) for _ in range(b)]
        scale = c / sum(w)
        sizes = [max(1, int(x * scale)) for x in w]
    else:
        shapes = {"mlp": lambda: ks.mlp_shapes(), "resnet18": lambda: ks.resnet18_shapes(num_classes=a),
                  "resnet50": lambda: ks.resnet50_shapes(num_classes=a),
                  "gpt2": lambda: ks.gpt2_small_shapes(n_layer=a, n_embd=b, vocab=c),
                  "llama": lambda: ks.llama_shapes(n_layer=a, hidden=b, ffn=b * 11 // 4, vocab=c)}[k]()
        sizes = [ks.numel(s) for s in shapes]
    return merge_small(sizes, case["block_min"]) if case["block_min"] else sizes


def _ratios(case):
    g = case["grid"]
    if g == "paper":
        return paper_grid().tolist()
    return ks.ratio_grid({"log16": -3, "log32": -4, "log64": -5}[g], 0, int(g[3:])).tolist()


def _budget(case):
    return int(case["budget"] * 4 * sum(_sizes(case)))


def _values(gen, n, dist, scale, out):
    """`n` values of the distribution into `out`.  Student's t by Bailey's polar method (Math. Comp. 62, 1994):
    sqrt(nu (u^(-2/nu) - 1)) cos(2 pi v) for uniform u, v."""
    dev = out.device
    if dist == "normal":
        out.copy_(torch.randn(n, generator=gen, device=dev).mul_(scale))
        return
    u = 1.0 - torch.rand(n, generator=gen, device=dev)
    v = torch.rand(n, generator=gen, device=dev)
    if dist == "laplace":
        out.copy_(u.log_().mul_(-scale).mul_(v.sub_(0.5).sign_()))
        return
    nu = float(dist[1:])
    t = u.pow_(-2.0 / nu).sub_(1.0).mul_(nu).sqrt_().mul_(v.mul_(2.0 * math.pi).cos_()).mul_(scale)
    if dist == "t2.5":
        # the outliers of the headline set: a thousandth of the entries a hundred times as large
        t = torch.where(torch.rand(n, generator=gen, device=dev) < 1e-3, t * 100.0, t)
    out.copy_(t)


def _flat(gen, sizes, scales, dist, factor=1.0, shift=0):
    """A flat buffer of the layers back to back, `shift` elements into its allocation."""
    out = torch.empty(sum(sizes) + shift, dtype=torch.float32, device="cuda")[shift:]
    at = 0
    for n, s in zip(sizes, scales):
        _values(gen, n, dist, factor * s, out[at:at + n])
        at += n
    return out


def prepare(case, seed):
    sizes = _sizes(case)
    d, L = sum(sizes), len(sizes)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    r = random.Random(seed)
    lo, hi = RECIPES[case["dist"]]
    scales = [10.0 ** r.uniform(lo, hi) for _ in sizes]
    if case["op"] == "server":
        starts = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
        starts[1:] = torch.cumsum(torch.tensor(sizes, dtype=torch.int64), 0).cuda()
        payloads, hats = [], []
        for _ in range(case["workers"]):
            # the payload of a worker: its share of the entries, at ascending places
            flat = torch.nonzero(torch.rand(d, generator=gen, device="cuda") < case["budget"] / 2).reshape(-1)
            layer = torch.searchsorted(starts, flat, right=True) - 1
            idx = (flat - starts[layer]).to(torch.int32)
            val = torch.randn(idx.numel(), generator=gen, device="cuda").mul_(1e-3)
            payloads.append((idx, val, torch.searchsorted(flat, starts)))
            hats.append(_flat(gen, sizes, scales, case["dist"]))
        x = torch.randn(d, generator=gen, device="cuda").mul_(0.02)
        return dict(op="server", d=d, starts=starts, payloads=payloads, hats=hats, x=x, weights=[1.0 / len(hats)] * len(hats),
                    status=torch.zeros(len(hats), dtype=torch.int32, device="cuda"))

    budget, ratios = _budget(case), _ratios(case)
    if case["h_factor"]:
        h = _flat(gen, sizes, scales, case["dist"], case["h_factor"], case["h_shift"])
    else:
        h = torch.zeros(d + case["h_shift"], dtype=torch.float32, device="cuda")[case["h_shift"]:]
    uniform = kimad.kimad_uniform_sizes(sizes, budget, _pair(case))[0] if case["op"] == "uniform" else None
    # with the dense fallback the payload may hold whole layers (their positions need not travel)
    capacity = d if case["dense"] else sum(uniform) if uniform else budget // _pair(case) + 1
    units = torch.cuda.get_device_properties(0).multi_processor_count
    plans = []
    for _ in range(2):
        g = _flat(gen, sizes, scales, case["dist"])
        p = kimad.Plan(g, h, sizes, ratios, D=case["D"], max_budget_bytes=budget,
                       cfg_flags=binding.KIMAD_CFG_DENSE_FALLBACK if case["dense"] else 0, capacity_pairs=capacity,
                       max_workgroups=units - 8 if case["op"] == "overlap" else 0,
                       value_format=binding.KIMAD_VALUES_F16 if case["f16"] else binding.KIMAD_VALUES_F32)
        p.idx.zero_()
        p.val.zero_()
        plans.append(p)
    state = dict(op=case["op"], h=h, plans=plans, budget=budget, turn=0)
    if uniform:
        K = torch.tensor(uniform, dtype=torch.int64)
        off = torch.zeros(L + 1, dtype=torch.int64)
        off[1:] = torch.cumsum(K, 0)
        state.update(K=K.cuda(), offsets=off.cuda())
    elif case["op"] == "overlap":
        state.update(side=torch.cuda.Stream(), done=[torch.cuda.Event() for _ in plans])
        for p, e in zip(plans, state["done"]):
            p.profile(budget_hint_bytes=budget)
            p.allocate(budget)
            e.record()
    for _ in plans:
        run(state)
    return state


def run(state):
    if state["op"] == "server":
        kimad.kimad_server_apply(state["payloads"], state["hats"], state["weights"], state["starts"], state["d"], state["x"],
                                 1e-3, status_out=state["status"])
        return [state["hats"], state["x"], state["status"]]
    turn = state["turn"]
    state["turn"] = 1 - turn
    p, other = state["plans"][turn], state["plans"][1 - turn]
    if state["op"] == "uniform":
        p.compress_ef(state["K"], state["offsets"])
        return [p.idx, p.val, p.status, state["h"]]
    if state["op"] == "step":
        p.step(state["budget"])
        return [p.err_table, p.j, p.K, p.offsets, p.status, p.idx, p.val, state["h"]]
    # this round is compressed with the sizes of the round before; its own are found on a second stream beside that
    main, side = torch.cuda.current_stream(), state["side"]
    p.profile(budget_hint_bytes=state["budget"])
    main.wait_event(state["done"][1 - turn])
    side.wait_stream(main)
    with torch.cuda.stream(side):
        p.allocate(state["budget"])
        state["done"][turn].record(side)
    p.compress_ef(other.K, other.offsets, reuse_profile=True)
    return [p.err_table, p.j, p.K, p.offsets, p.status, p.idx, p.val, state["h"]]


def work(case):
    sizes = _sizes(case)
    d, L = sum(sizes), len(sizes)
    if case["op"] == "server":
        M, pairs = case["workers"], case["budget"] / 2 * d
        # decode: pairs read, their estimator entries read and written; step: estimators and model read, model written
        return {"bytes": M * pairs * 16 + 4 * (M + 2) * d, "flops": M * pairs + (2 * M + 2) * d}
    pair = _pair(case)
    pairs = min(d, _budget(case) // pair)
    J = len(_ratios(case))
    # g and h read once, payload written, its estimator entries written; the table and the sizes
    small = 8 * L * (J + 3) if case["op"] != "uniform" else 16 * L
    return {"bytes": 8 * d + pairs * (pair + 4) + small, "flops": 3 * d}


def tolerance(case):
    if case["op"] in ("uniform", "server"):
        return "exact"          # a selection, single fp32 additions, and fp64 sums in a fixed order
    # Whole numbers, payload and estimator are exact.  The error table's sums are of squares cut to 24 bits with bounds
    # on what is cut: against fp64 sums over a sorted layer it is off by 5e-9 to 9e-9 in the 2-norm (ResNet-50,
    # ResNet-18 on the paper's grid, perceptron; 8e-7 for a single entry).
    return {"rel": 4e-8}
