"""The optimizer step as users of this package run it: one pass = one `AdaPM.step` over a whole block table.

A case is a transformer-shaped block table (the tables of `workloads.py`, spelled out in numbers), the dtypes of its
parameters and gradients, the refresh period T and the kind of step that is timed:

  step = "alg2"   a step that runs Alg. 2 (with T = 1 the literal Alg. 1, every step of such a run; with T > 1 the step
                  on the refresh grid, followed by the orthonormalisation of R);
  step = "held"   a step between two refreshes (T > 1): 99 of 100 steps of a run with T = 100.

Parameters and gradients live in one flat buffer each, as bucketed training programs keep them; the optimizer state and
workspace belong to the `AdaPM` object.  A pass updates parameters and state in place and returns them.
"""
import math

import torch

from paper_2510_09103_amd.optimizer import AdaPM, make_hparams
from paper_2510_09103_amd.workloads import BlockSpec

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
_LR = 1e-3
_WARM_STEPS = 2        # steps before the first timed one, each on another gradient of the same slowly moving subspace


def _case(name, d, ffn, layers, rank, *, gated=False, vocab=0, positions=0, untied=False, head=64, regimes="matrices",
          v="element", params="bf16", grads="bf16", T=1, step="alg2", clip=0.0):
    return dict(name=name, d=d, ffn=ffn, layers=layers, rank=rank, gated=gated, vocab=vocab, positions=positions, untied=untied,
                head=head, regimes=regimes, v=v, params=params, grads=grads, T=T, step=step, clip=clip)


def listed():
    # one transformer block in fp32, nine tensors of at most 1 MB: a unit test, a toy model, a fine-tuned adapter.  The
    # arithmetic is nothing, launches and latencies are everything.
    tiny = dict(d=256, ffn=1024, layers=1, rank=8, gated=True, params="f32", grads="f32")
    # 42 M parameters kept in fp32 with bf16 gradients: the exact (fp64) contractions, small-model research
    m60 = dict(d=512, ffn=1376, layers=8, rank=32, gated=True, vocab=32000, params="f32", grads="bf16")
    # 355 M parameters in bf16, per-element second moment: an ordinary pre-training run on one GPU
    m350 = dict(d=1024, ffn=4096, layers=24, rank=64, vocab=50304, positions=1024)
    # 1.34 B parameters, per-element second moment, an MLP width that is no multiple of anything (5461): ragged rows and
    # columns in a third of the gradients each; the paper's runs clip the global gradient norm
    m1b = dict(d=2048, ffn=5461, layers=24, rank=128, gated=True, vocab=32000, untied=True, head=128)
    # 1.64 B parameters, blockwise second moment, rank 128 on every layer matrix: the benchmark's table, the largest here
    m15b = dict(d=1600, ffn=6400, layers=48, rank=128, vocab=50257, positions=1024, untied=True, v="blockwise")
    # the paper's own assignment of momentum regimes on its 350 M shape (no momentum on embeddings and output projections,
    # full momentum on values, rank 5 % = 51 elsewhere), with the global clipping of the paper's runs
    paper = dict(d=1024, ffn=2736, layers=24, rank=0, gated=True, vocab=32000, regimes="paper", clip=1.0)
    return [
        _case("tiny_literal", **tiny),
        _case("tiny_held", **tiny, T=100, step="held"),
        _case("60m_f32_literal", **m60),
        _case("60m_f32_held", **m60, T=100, step="held"),
        _case("350m_literal", **m350),
        _case("350m_held", **m350, T=100, step="held"),
        _case("350m_paper_held_clip", **paper, T=100, step="held"),
        _case("1b_ragged_literal_clip", **m1b, clip=1.0),
        _case("1b_ragged_held", **m1b, T=100, step="held"),
        _case("1.5b_literal", **m15b),
        _case("1.5b_held", **m15b, T=100, step="held"),
        _case("1.5b_refresh", **m15b, T=100, step="alg2"),
    ]


def draw(rng):
    """Another model of the same ranges: widths 64 .. 2048 (multiples of 64, of 8, or odd), 1 .. 48 layers, plain or gated
    MLPs, any rank up to 128, with and without embeddings, either second moment, either regime table, either kind of step."""
    d = round(64 * 32 ** rng.random())
    shape = rng.random()
    if shape < 0.5:
        d = 64 * max(1, round(d / 64))
    elif shape < 0.85:
        d = 8 * round(d / 8)
    head = rng.choice([h for h in (32, 64, 128) if d % h == 0] or [0])
    gated = rng.random() < 0.5
    ffn = 4 * d if not gated else round(8 * d / 3)
    f32 = rng.random() < 0.3
    T, step = rng.choice([(1, "alg2"), (100, "held"), (100, "held"), (100, "alg2")])
    c = _case("", d, ffn, round(48 ** rng.random()), min(d, rng.choice([0, round(4 * 32 ** rng.random()), 32, 64, 128])),
              gated=gated, vocab=rng.choice([0, round(1000 * 50 ** rng.random())]), positions=rng.choice([0, 1024]),
              untied=rng.random() < 0.3, head=head, regimes=rng.choice(["matrices", "matrices", "paper"]),
              v=rng.choice(["element", "blockwise"]), params="f32" if f32 else "bf16",
              grads=rng.choice(["f32", "bf16"]) if f32 else "bf16", T=T, step=step, clip=rng.choice([0.0, 0.0, 1.0]))
    del c["name"]
    # no more than the largest listed case: fewer layers where the model would be larger (the exact contractions of fp32
    # parameters cost about two hundred times as much per operation as the split-bf16 ones)
    while c["layers"] > 1:
        w, n = work(c), sum(b.numel for b in _table(c))
        if n <= 7e8 and (not f32 or w["flops"] <= 5e10):
            break
        c["layers"] -= 1
    return c


def _table(c):
    """The block table of a case: the same blocks, in the same order, as the tables of `workloads.py`."""
    d, f, gd, pd = c["d"], c["ffn"], c["grads"], c["params"]
    paper, mini = c["regimes"] == "paper", c["v"] == "blockwise"
    heads = c["head"] if mini and c["head"] else 1
    rows = dict(v_mode="rowgroup") if mini else {}

    def lowrank(name, m, n, group=1):
        r = c["rank"] or max(1, round(0.05 * min(m, n)))
        return BlockSpec(name, m, n, pd, gd, "lowrank", r, weight_decay=0.1, **(dict(rows, v_group_rows=group) if mini else {}))

    def dense(name, m, n, mom, wd=0.1):
        return BlockSpec(name, m, n, pd, gd, mom, 0, lr_scale=0.75 if mom == "none" else 1.0, weight_decay=wd, **rows)

    def norm(name):
        return BlockSpec(name, d, 1, pd, gd, "full", 0, "whole" if mini else "element", is_norm=True)

    table = []
    if c["vocab"]:
        table.append(dense("embed", c["vocab"], d, "none" if paper else "full"))
        if c["positions"]:
            table.append(dense("pos", c["positions"], d, "none" if paper else "full"))
    for k in range(c["layers"]):
        table += [lowrank(f"l{k}.q", d, d, heads), lowrank(f"l{k}.k", d, d, heads)]
        if paper:
            table += [dense(f"l{k}.v", d, d, "full"), dense(f"l{k}.o", d, d, "none")]
        else:
            table += [lowrank(f"l{k}.v", d, d), lowrank(f"l{k}.o", d, d)]
        table += [lowrank(f"l{k}.{n}", f, d) for n in (("gate", "up") if c["gated"] else ("up",))]
        table += [lowrank(f"l{k}.down", d, f), norm(f"l{k}.n1"), norm(f"l{k}.n2")]
    if c["vocab"]:
        table.append(norm("n_f"))
        if c["untied"]:
            table.append(dense("out", c["vocab"], d, "none" if paper else "full"))
    return table


def _flat(table, dtype):
    """One buffer for the whole table and its blocks as views of it (every block starts on a whole 128 bytes)."""
    at, n = [], 0
    for b in table:
        at.append(n)
        n += (b.numel + 63) // 64 * 64
    flat = torch.zeros(n, dtype=dtype, device="cuda")
    return flat, [flat[o:o + b.numel].view(b.rows, b.cols) for o, b in zip(at, table)]


def prepare(case, seed):
    table = _table(case)
    gen = torch.Generator("cuda").manual_seed(seed)

    def randn(*size):
        return torch.randn(*size, device="cuda", generator=gen)

    params_flat, params = _flat(table, _DT[case["params"]])
    _, grads = _flat(table, _DT[case["grads"]])
    for b, w in zip(table, params):
        if b.is_norm:
            w.fill_(1.0)
        else:
            w.copy_(randn(b.rows, b.cols).mul_(0.02))
    # what transformer gradients look like (workloads.py): a decaying spectrum on a fixed subspace whose weights move
    # from step to step, and noise
    bases = []
    for b in table:
        k = min(128, b.rows, b.cols)
        bases.append(None if b.cols == 1 else (randn(b.rows, k).div_(math.sqrt(b.rows)), randn(k, b.cols).div_(math.sqrt(b.cols)),
                                               torch.arange(1, k + 1, device="cuda", dtype=torch.float32) ** -1.5, randn(k)))

    def gradients():
        for b, g, basis in zip(table, grads, bases):
            if basis is None:
                g.copy_(randn(b.rows, 1).mul_(1e-2))
            else:
                u, v, s, a = basis
                a.mul_(0.9).add_(randn(a.numel()), alpha=math.sqrt(1 - 0.81))
                g.copy_(torch.addmm(randn(b.rows, b.cols), u * (s * a.clamp(-2, 2)), v, beta=1e-4))

    opt = AdaPM(table, make_hparams(T=case["T"]), grad_clip=case["clip"])
    for t in range(1, _WARM_STEPS + 1):
        gradients()
        opt.step(params, grads, t, _LR)
    gradients()
    out = {"params": params_flat, "state": opt.state.view(torch.float32)}
    # the whole flat buffers, and besides one block of every kind for itself, whose factors, momentum and second moment
    # differ in scale by many orders of magnitude
    seen = set()
    for i, b in enumerate(table):
        kind = (b.rows, b.cols, b.mom, b.v_mode, b.v_group_rows)
        if kind not in seen and len(seen) < 10:
            seen.add(kind)
            out[f"{b.name}.W"] = params[i]
            out.update({f"{b.name}.{k}": x for k, x in opt.state_view(i).items()})
    return {"opt": opt, "params": params, "grads": grads, "passes": 0, "T": case["T"], "step": case["step"], "out": out}


def run(state):
    # step numbers as a training loop counts them, of the kind that the case times
    i, T = state["passes"], state["T"]
    state["passes"] += 1
    if T == 1:
        t = _WARM_STEPS + 1 + i
    elif state["step"] == "alg2":
        t = T * (i + 1) + 1
    else:
        t = _WARM_STEPS + 1 + i % (T - _WARM_STEPS)
    state["opt"].step(state["params"], state["grads"], t, _LR)
    return state["out"]


def work(case):
    size = {"f32": 4, "bf16": 2}
    alg2 = case["step"] == "alg2"
    nbytes = flops = 0
    for b in _table(case):
        m, n, r, mn = b.rows, b.cols, b.rank, b.numel
        # gradient in, parameter in and out, second moment in and out
        nbytes += mn * (size[b.grad_dtype] + 2 * size[b.param_dtype])
        nbytes += 8 * (mn if b.v_mode == "element" else m // b.v_group_rows if b.v_mode == "rowgroup" else 1)
        if b.mom == "full":
            nbytes += 8 * mn
        elif b.mom == "lowrank":
            # both factors in and out, four effective iterations of two products with G and the thin ones, then the rank-2r
            # term of the bias correction; with R held only L is written, one product with G and one of rank r
            nbytes += 8 * (m + n) * r if alg2 else 8 * m * r + 4 * n * r
            flops += 4 * (4 * mn * r + 8 * r * r * (m + n)) + 4 * mn * r if alg2 else 4 * mn * r
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["params"] == "f32":
        # contractions in fp64, everything else in fp32
        return {"rel": 1e-5, "max": 4e-4}
    # Contractions on split-bf16 operands with fp32 sums.  Against the same cases with the contractions in fp64 the outputs
    # of one and two passes differ by at most 7e-5 (2-norm, the worst block of any case: its bf16 parameters, of which some
    # on a rounding boundary fall to either side) and 1.6e-2 (two such roundings in one element); four times that is allowed.
    return {"rel": 3e-4, "max": 0.06}
