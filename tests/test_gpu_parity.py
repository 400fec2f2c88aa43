"""GPU parity: the HIP library against the CPU oracle, element by element, on the same
seeded inputs.  Tolerances (relative, per element, with a block-RMS floor):
  TOL32   1e-5  fp32 parameters and their state on the exact (fp64) contraction path;
  TOLX    2e-4  fp32 parameters and any state on the split-bf16 MFMA path, runs of up to 20 steps (worst seen 1.1e-4);
  TOLX_LONG 4e-3  the same over 50 - 100 steps.  Alg. 2 is a warm-started iteration whose state is carried from step
                to step, and it amplifies perturbations: rounding the ORACLE's own state to fp32 once per step
                (6e-8) already moves its product L R by 4e-5 after 100 steps.  The MFMA path perturbs every step
                by ~1e-6 (fp32 accumulation, operands split to 2^-17), so its distance from the oracle grows with
                the step count: product L R of config 3 1e-4 after 20 steps, 2e-4 after 30, 2.2e-3 after 100
                (bound: twice that); the exact (fp64) contraction path stays at 5e-6 (config 2, and config 3's
                strata re-run on it below);
  bf16 parameters: 2e-3 or a bounded number of representable values, with asserted flip fractions
                (parity_util.compare_params)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import adapm_oracle as O
from paper_2510_09103_amd import binding as B
from paper_2510_09103_amd import workloads as WL
from paper_2510_09103_amd.workloads import BlockSpec
from parity_util import Pair, to_np

pytestmark = pytest.mark.gpu

TOL32 = 1e-5
TOLX = 2e-4
TOLX_LONG = 4e-3
TOL16 = TOLX      # state and fp32 parameters of runs on the MFMA path


def run(wl, steps, hp=None, tol_state=TOL32, tol_param=TOL32, check_every=None, **kw):
    pair = Pair(wl, hp, **kw)
    pair.flip_per_step = max(pair.flip_per_step, 10.0 * tol_state)
    rep = None
    for t in range(1, steps + 1):
        pair.step()
        if check_every and t % check_every == 0:
            rep = pair.compare(tol_state, tol_param)
    rep = pair.compare(tol_state, tol_param)
    print(f"{wl.name} hp={hp} steps={steps}: {rep}", flush=True)
    return pair, rep


def test_seeded_start_is_bit_identical():
    wl = WL.subset(WL.llama_60m(), ["l0.attn.q", "l0.ffn.down"])
    pair = Pair(wl, dict(seed=12345))
    for i in range(2):
        sv = pair.opt.state_view(i)
        assert np.array_equal(sv["R"].cpu().numpy(), pair.state_o[i]["R"])
        assert float(sv["L"].abs().max()) == 0.0 and float(sv["v"].abs().max()) == 0.0
    pair0 = Pair(wl, dict(seed=0))
    assert float(pair0.opt.state_view(0)["R"].abs().max()) == 0.0


@pytest.mark.parametrize("T", [1, 4])
def test_config1_tiny_block(T):
    run(WL.tiny_block(), 10, dict(T=T), check_every=1)


def mixed_table(pd="f32", gd="f32"):
    mk = BlockSpec
    return WL.Workload("mixed", (
        mk("none_mat", 100, 37, pd, gd, "none", 0, "element", 1, 0.75, 0.1),
        mk("full_rg3", 129, 67, "bf16", "bf16", "full", 0, "rowgroup", 3, 1.0, 0.1),
        mk("vec_whole", 1000, 1, pd, "bf16", "full", 0, "whole", 1, 1.0, 0.0),
        mk("lr_ragged", 200, 131, pd, gd, "lowrank", 5, "rowgroup", 1, 1.0, 0.1),
        mk("lr_heads", 96, 160, "bf16", "bf16", "lowrank", 16, "rowgroup", 32, 1.0, 0.1, 32),
        mk("full_whole_big", 300, 200, pd, gd, "full", 0, "whole", 1, 1.0, 0.05),
        mk("lr_fullrank_wide", 64, 1000, pd, "bf16", "lowrank", 64, "element", 1, 1.0, 0.1),
        mk("one", 1, 1, pd, gd, "full", 0, "element", 1, 1.0, 0.0),
        mk("none_vec", 77, 1, pd, gd, "none", 0, "rowgroup", 7, 0.75, 0.0),
        mk("lr_rank1", 70, 66, pd, gd, "lowrank", 1, "whole", 1, 1.0, 0.1),
    ), steps=6, seed=3, signal_rank=24)


@pytest.mark.parametrize("hp", [
    dict(T=1), dict(T=3), dict(T=1, adam_debias=1, clip=float("inf")), dict(T=2, bias_correction=0),
    dict(T=1, bias_correction=0, K=3), dict(T=1, K=1), dict(T=2, K=1), dict(T=1, beta1=0.0),
])
def test_mixed_table_all_modes(hp):
    wl = mixed_table()
    # every mode on the exact (fp64 contraction) path at the fp32 tolerance; the MFMA path has its own
    # tables below.  bf16-parameter blocks are held to the bf16 criterion inside compare_params
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_F64)
    run(wl, 6, hp, tol_state=TOL32, tol_param=TOL32, check_every=2)


def ragged_bf16_table():
    """bf16 blocks on the MFMA path whose sizes are not multiples of the 128- and 256-row stripes, the 64-column chunks
    or the 8-element vectors; every rank class; every kind of v."""
    mk = BlockSpec
    return WL.Workload("ragged_bf16", (
        mk("r32_cols1000", 200, 1000, "bf16", "bf16", "lowrank", 32, "rowgroup", 1, 1.0, 0.1),
        mk("r64_small", 96, 136, "bf16", "bf16", "lowrank", 64, "element", 1, 1.0, 0.1),
        mk("r128_rows130", 130, 264, "bf16", "bf16", "lowrank", 128, "rowgroup", 65, 1.0, 0.1),
        mk("r32_f32params", 70, 72, "f32", "bf16", "lowrank", 32, "whole", 1, 1.0, 0.0),
        mk("r64_heads16", 192, 320, "bf16", "bf16", "lowrank", 64, "rowgroup", 16, 1.0, 0.1, 16),
        # columns that are not a multiple of 8: rows of G, W and v start at any 2-byte (4-byte) alignment and the
        # last cols mod 8 columns of every row are done element by element
        mk("r32_cols1001", 200, 1001, "bf16", "bf16", "lowrank", 32, "rowgroup", 1, 1.0, 0.1),
        mk("r64_cols77_elem", 96, 77, "bf16", "bf16", "lowrank", 64, "element", 1, 1.0, 0.1),
        mk("r128_cols333_f32params", 136, 333, "f32", "bf16", "lowrank", 128, "element", 1, 1.0, 0.0),
        mk("r32_cols70_whole", 130, 70, "bf16", "bf16", "lowrank", 20, "whole", 1, 1.0, 0.1),
    ), steps=6, seed=5, signal_rank=40)


@pytest.mark.parametrize("hp", [
    dict(T=1), dict(T=3), dict(T=2, bias_correction=0), dict(T=1, adam_debias=1, clip=float("inf")),
    dict(T=2, K=1), dict(T=1, beta1=0.0),
])
def test_ragged_shapes_on_the_mfma_path(hp):
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2)
    run(ragged_bf16_table(), 6, hp, tol_state=TOL16, tol_param=TOL16, check_every=2)


@pytest.mark.parametrize("first", [1, 4])
@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_every_row_remainder_in_the_stripe_products(first, hp):
    """Row lengths of every remainder mod 8 (and so mod 4), below one vector's width past a 64-column chunk and past a
    256-column stripe: the columns behind a row's last whole vector join the products, and the sums of squares of the
    per-row second moment, behind the loops, and the rows of R are stored at 4-byte alignments."""
    wl = WL.Workload("remainders", tuple(
        BlockSpec(f"c{c}_r{r}", 70 + c % 7, c, "bf16", "bf16", "lowrank", r, v, 1, 1.0, 0.1)
        for r, v, base in ((8, "rowgroup", 8), (40, "element", 64), (70, "rowgroup", 256), (32, "whole", 512 + 56))
        for c in range(base + first, base + first + 4)), steps=4, seed=9, signal_rank=8)
    run(wl, 4, dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOL16, tol_param=TOL16, check_every=2)


@pytest.mark.parametrize("hp", [dict(K=1), dict(K=2), dict(K=3), dict(K=1, bias_correction=0), dict(K=2, T=2)])
def test_factors_that_reach_the_state_without_a_copy(hp):
    """Where rows are whole vectors the last iteration's stripes write R over the old one, elsewhere it is copied; L is written
    by the update, which reads the old one.  Stripes that end inside, at and past a chunk, ranks that are no multiple of 4."""
    wl = WL.Workload("stored", tuple(
        BlockSpec(f"{m}x{n}_r{r}", m, n, "bf16", "bf16", "lowrank", r, v, 1, 1.0, 0.1)
        for m, n, r, v in ((70, 8, 5, "element"), (128, 64, 32, "rowgroup"), (129, 264, 70, "whole"), (257, 520, 128, "element"),
                           (136, 263, 64, "rowgroup"), (40, 256, 33, "rowgroup"))), steps=4, seed=23, signal_rank=8)
    run(wl, 4, dict(dict(T=1, contraction=B.ADAPM_CONTRACT_BF16X2), **hp), tol_state=TOL16, tol_param=TOL16, check_every=1)


@pytest.mark.parametrize("groups", [1, 5, 8189, 8190, 8193, 20000])
def test_groups_dealt_to_workgroups(groups):
    """Few groups are spread over the chip, four to a workgroup, more of them where there are many: counts at which the share
    of a workgroup changes (the smaller block adds three), and last workgroups with one group."""
    wl = WL.Workload("dealt", (
        BlockSpec("rows", groups, 16, "bf16", "bf16", "full", 0, "rowgroup", 1, 1.0, 0.1),
        BlockSpec("wide", 3, 2048, "bf16", "bf16", "none", 0, "rowgroup", 1, 1.0, 0.1)), steps=2, seed=31)
    run(wl, 2, dict(T=1), tol_state=TOL16, tol_param=TOL16, check_every=1)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_rows_a_multiple_of_the_chunks_with_ragged_columns(hp):
    """The other end of a gradient whose rows are no whole vectors: rows that fill the last chunk of the transposed product
    exactly (64), or all but one of it, with odd columns, so that its very last element sits alone in its dword."""
    wl = WL.Workload("whole_chunks", tuple(
        BlockSpec(f"{m}x{n}_r{r}", m, n, "bf16", "bf16", "lowrank", r, v, 1, 1.0, 0.1)
        for m, n, r, v in ((64, 73, 8, "element"), (128, 331, 40, "rowgroup"), (192, 515, 70, "element"), (256, 257, 128, "whole"),
                           (63, 513, 32, "rowgroup"), (320, 9, 4, "element"))), steps=4, seed=19, signal_rank=8)
    pair, _ = run(wl, 4, dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOL16, tol_param=TOL16, check_every=2)
    labels = labels_of_a_step(pair.opt, pair.params, pair.stream.next(), 1, pair.wl.lr)
    assert "alg2_stripe_step_r128" in labels and "alg2_products_mfma" not in labels, labels


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_both_contraction_paths_in_one_table(hp):
    """Automatic choice of the contraction: the fp32-parameter blocks of the table take the exact path, the bf16 ones
    the MFMA path.  With T > 1 the exact path's step with R held needs scratch in every step while the MFMA path's
    bf16 copies of R have to survive beside it (the layout that may not put the one over the other)."""
    run(ragged_bf16_table(), 6, dict(hp), tol_state=TOL16, tol_param=TOL16, check_every=2)


def labels_of_a_step(opt, params, grads, t, lr):
    """kernel classes that one step of this optimizer launches"""
    torch.cuda.synchronize()
    B.adapm_profile_read(opt.ctx)
    B.adapm_profile_enable(opt.ctx, True)
    opt.step(params, grads, t, lr)
    torch.cuda.synchronize()
    labels = set(B.adapm_profile_read(opt.ctx))
    B.adapm_profile_enable(opt.ctx, False)
    return labels


def long_ragged_table():
    """Long blocks whose rows are no whole vectors and whose rank is small for their size: the fragment images that stripe
    products need would outgrow the scratch (30 MiB here, the state is smaller than that), so Alg. 2 runs as split-bf16 GEMMs.
    Tall and wide, every rank class, every kind of v, both types of parameters; the contractions over the long side walk
    up to 4096 chunks, with a remainder."""
    mk = BlockSpec
    return WL.Workload("long_ragged", (
        mk("tall_r1", 131072, 9, "bf16", "bf16", "lowrank", 1, "element", 1, 1.0, 0.1),
        mk("wide_r5", 9, 70001, "bf16", "bf16", "lowrank", 5, "rowgroup", 3, 1.0, 0.1),
        mk("tall_r40_f32params", 40001, 75, "f32", "bf16", "lowrank", 40, "whole", 1, 1.0, 0.0),
        mk("tall_r100", 20003, 130, "bf16", "bf16", "lowrank", 100, "rowgroup", 1, 1.0, 0.1),
    ), steps=4, seed=15, signal_rank=8)


@pytest.mark.parametrize("hp,clip", [(dict(T=1), None), (dict(T=3), None), (dict(T=1, normalise=1), None), (dict(T=2, bias_correction=0), 0.5)])
def test_long_ragged_blocks_on_the_split_gemms(hp, clip):
    pair, _ = run(long_ragged_table(), 3, dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOL16, tol_param=TOL16,
                  grad_clip=clip)
    labels = labels_of_a_step(pair.opt, pair.params, pair.stream.next(), 1, pair.wl.lr)
    assert {"alg2_products_mfma", "alg2_update_mfma"} <= labels, labels
    assert not any(l.startswith("alg2_stripe") for l in labels), labels
    assert ("alg2_step_normaliser" in labels) == bool(hp.get("normalise"))


def exact_edges_table(gd, many):
    """Blocks of the exact path at the edges of its output tiles (16 and 32 wide), of the steps of the contraction (16 and
    32 long) and of the two-column loads: ranks around 16, 32 and 128, sizes one beside a multiple; many: enough Gram
    matrices for the larger of their two tile shapes (1024 tiles of 32 x 32 over four matrices of every block)."""
    mk = BlockSpec
    if many:
        sizes = [(131, 129, 128)] * 15 + [(129, 200, 127)] * 2
    else:
        sizes = [(2, 2, 1), (3, 2, 2), (17, 33, 1), (15, 16, 15), (16, 48, 16), (33, 17, 17), (31, 65, 16), (64, 31, 31),
                 (32, 64, 32), (97, 63, 33), (140, 150, 129)]
    return WL.Workload("exact_edges", tuple(mk(f"b{i}_{m}x{n}_r{r}", m, n, "f32", gd, "lowrank", r, "element", 1, 1.0, 0.1)
                                            for i, (m, n, r) in enumerate(sizes)), steps=4, seed=31, signal_rank=24)


@pytest.mark.parametrize("gd,many", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("T", [1, 2])
def test_exact_path_at_the_edges_of_its_tiles(gd, many, T):
    """fp64 contractions with every intermediate in fp64: the fp32 tolerance (state rounded once per step)."""
    run(exact_edges_table(gd, many), 4, dict(T=T), tol_state=TOL32, tol_param=TOL32)


@pytest.mark.parametrize("copies", [1, 12, 30])
@pytest.mark.parametrize("hp", [dict(T=1), dict(T=2), dict(T=1, K=2), dict(T=1, K=3, normalise=1)])
def test_exact_path_for_every_number_of_waves_on_a_tile(copies, hp):
    """Launches of few output tiles split a contraction over 8 waves, the others over 4 and may deal whole blocks to an XCD;
    with two GD iterations or more the last one writes the factors to the state, with one (K = 2) a launch of its own.  Sums in
    fp64 whatever the split: the fp32 tolerance."""
    sizes = [(17, 33, 1), (33, 17, 17), (64, 31, 31), (97, 63, 33)]
    wl = WL.Workload("exact_waves", tuple(BlockSpec(f"b{k}_{m}x{n}_r{r}", m, n, "f32", "bf16" if k % 2 else "f32", "lowrank", r, "element", 1, 1.0, 0.1)
                                          for k in range(copies) for m, n, r in sizes), steps=3, seed=43, signal_rank=24)
    run(wl, 3, hp, tol_state=TOL32, tol_param=TOL32)


@pytest.mark.parametrize("v", ["element", "rowgroup"])
@pytest.mark.parametrize("hp", [dict(T=1), dict(T=2)])
def test_exact_path_at_ranks_whose_factors_pass_the_lds_of_the_update(hp, v):
    """The update stages 128 values of k of a factor at a time: one less and one more, and second and third shares of whole steps with
    and without an edge, in the kernel of one type and in the one of several."""
    sizes = [(140, 150, 127), (140, 150, 129), (150, 210, 144), (210, 263, 200), (300, 280, 272)]
    for types in (["f32"], ["f32", "bf16"]):
        wl = WL.Workload("wide", tuple(BlockSpec(f"b{k}_{m}x{n}_r{r}", m, n, "f32", types[k % len(types)], "lowrank", r, v, 1, 1.0, 0.1)
                                       for k, (m, n, r) in enumerate(sizes)), steps=2, seed=61, signal_rank=24)
        run(wl, 2, hp, tol_state=TOL32, tol_param=TOL32)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=2)])
@pytest.mark.parametrize("gd", ["f32", "bf16"])
def test_exact_path_without_requests_ahead(gd, hp):
    """Launches that fill the chip several times load the operands of a step where they use them: contractions of less than a step, of
    whole steps and beside them, shares of one to seven steps per wave."""
    sizes = [(16, 48, 8), (17, 33, 15), (64, 15, 15), (97, 63, 33), (130, 112, 64), (48, 130, 17)]
    wl = WL.Workload("filled", tuple(BlockSpec(f"b{k}_{m}x{n}_r{r}", m, n, "f32", gd, "lowrank", r, "element", 1, 1.0, 0.1)
                                     for k in range(24) for m, n, r in sizes), steps=2, seed=59, signal_rank=24)
    run(wl, 2, hp, tol_state=TOL32, tol_param=TOL32)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=2)])
def test_every_type_of_block_in_one_update_of_the_exact_path(hp):
    """Both types of G and W, both kinds of second moment and blocks of fewer columns than a lane updates, in one launch of few tiles:
    sizes at and beside the edges of a tile, ranks whose factors fit the launch's LDS, fill it and pass it."""
    sizes = [(64, 64, 8), (65, 63, 31), (130, 67, 65), (97, 200, 70), (63, 129, 16), (33, 2, 2), (129, 3, 3), (16, 4, 4)]
    kinds = [(pd, gd, v) for pd in ("f32", "bf16") for gd in ("f32", "bf16") for v in ("element", "rowgroup")]
    wl = WL.Workload("types", tuple(BlockSpec(f"b{k}_{m}x{n}_r{r}", m, n, pd, gd, "lowrank", min(r, m, n), v, 1, 1.0, 0.1)
                                    for k, (m, n, r) in enumerate(sizes) for pd, gd, v in kinds[k % 2::2]), steps=3, seed=53, signal_rank=24)
    run(wl, 3, dict(hp, contraction=B.ADAPM_CONTRACT_F64), tol_state=TOL32, tol_param=TOL32)


@pytest.mark.parametrize("pd,gd,vm,clip", [("f32", "bf16", "element", None), ("bf16", "f32", "rowgroup", 0.5), ("bf16", "bf16", "element", None),
                                           ("f32", "f32", "whole", None)])
@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3), dict(T=2, bias_correction=0), dict(T=2, K=1)])
def test_update_of_the_exact_path_at_the_edges_of_its_tiles(pd, gd, vm, clip, hp):
    """Tiles of 64 x 64 with four columns per lane and steps of 16 along the rank: rows of 2 and 3 columns, one column beside
    a multiple of 4 and 64, rows beside a multiple of 16 and 64, ranks beside a multiple of 4 and 16; both types of G and W."""
    sizes = [(2, 2, 2), (5, 3, 3), (15, 4, 4), (16, 5, 1), (17, 63, 15), (63, 64, 16), (64, 65, 17), (65, 66, 5), (130, 131, 33)]
    wl = WL.Workload("update64_edges", tuple(BlockSpec(f"b{m}x{n}_r{r}", m, n, pd, gd, "lowrank", r, vm, 1, 1.0, 0.1)
                                             for m, n, r in sizes), steps=4, seed=41, signal_rank=24)
    run(wl, 4, dict(hp, contraction=B.ADAPM_CONTRACT_F64), tol_state=TOL32, tol_param=TOL32, grad_clip=clip)


def odd_rank_table():
    """bf16 blocks whose rank is not 32, 64 or 128 (the paper takes r = 5 % of the smaller dimension): the
    MFMA kernels run them in the next rank class with zero-padded images of the factors.  Ranks that are
    and are not multiples of 4 (vector / scalar access to the rows of L)."""
    mk = BlockSpec
    return WL.Workload("odd_ranks", (
        mk("r8", 136, 200, "bf16", "bf16", "lowrank", 8, "rowgroup", 1, 1.0, 0.1),
        mk("r20_rows130", 130, 264, "bf16", "bf16", "lowrank", 20, "element", 1, 1.0, 0.1),
        mk("r51", 264, 1024, "bf16", "bf16", "lowrank", 51, "rowgroup", 1, 1.0, 0.1),
        mk("r80_f32params", 160, 320, "f32", "bf16", "lowrank", 80, "whole", 1, 1.0, 0.0),
        mk("r100", 256, 136, "bf16", "bf16", "lowrank", 100, "rowgroup", 64, 1.0, 0.1),
    ), steps=6, seed=9, signal_rank=40)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_ranks_between_the_classes_on_the_mfma_path(hp):
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2)
    run(odd_rank_table(), 6, hp, tol_state=TOL16, tol_param=TOL16, check_every=2)


@pytest.mark.parametrize("ranks", [(1, 15, 16, 17, 31, 33), (47, 49, 64, 65, 80), (81, 93, 96, 97, 112), (113, 127, 128)])
def test_orthonormalisation_for_every_number_of_rank_steps(ranks):
    """R <- C^-1 R and L <- L C run in one body per number of 16-wide steps of the rank: first, last and middle ranks of each,
    columns and rows beside a multiple of 16 and 64.  Rows of R orthonormal to fp32 rounding (the sum of n products of values
    rounded to 2^-24, n |R_ik R_jk| <= 1 by Cauchy-Schwarz, on either side: 2 * 2^-24, times 4), and the product L R that of
    the same step without it (each factor rounded once more, r-term sums: 1e-6 in the 2-norm)."""
    blocks = [BlockSpec(f"r{r}", 145 + i, 208 + 13 * i, "bf16", "bf16", "lowrank", r, "rowgroup", 1, 1.0, 0.1) for i, r in enumerate(ranks)]
    got = {}
    for T in (1, 3):
        pair = Pair(WL.Workload("regauge", tuple(blocks), steps=1, seed=51, signal_rank=24),
                    dict(T=T, contraction=B.ADAPM_CONTRACT_BF16X2))
        pair.step()
        torch.cuda.synchronize()
        got[T] = [{k: v.double().cpu() for k, v in pair.opt.state_view(i).items()} for i in range(len(blocks))]
    for b, plain, ortho in zip(blocks, got[1], got[3]):
        eye = torch.eye(b.rank, dtype=torch.float64)
        assert float((ortho["R"] @ ortho["R"].T - eye).abs().max()) <= 8 * 2.0 ** -24, b.name
        want = plain["L"] @ plain["R"]
        assert float((ortho["L"] @ ortho["R"] - want).norm()) <= 1e-6 * float(want.norm()), b.name


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=2), dict(T=1, normalise=1)])
def test_sums_of_gram_segments_in_every_rank_class(hp):
    """Contractions of more than 25 chunks of 64 columns are cut into segments whose partial r x r sums a second launch adds, 16
    rows to a workgroup: ranks inside, at the end of and beyond a group of 16 rows and a chunk, in all three rank classes."""
    wl = WL.Workload("gram_segments", tuple(BlockSpec(f"b{m}x{n}_r{r}", m, n, "bf16", "bf16", "lowrank", r, "element", 1, 1.0, 0.1)
                                            for m, n, r in [(136, 1704, 15), (1701, 72, 32), (72, 1664, 33), (136, 1704, 64), (136, 1800, 65), (1668, 136, 113),
                                                            (136, 3304, 128)]), steps=3, seed=47, signal_rank=24)
    run(wl, 3, hp, tol_state=TOLX, tol_param=TOLX)


def random_table(rng, case):
    """A few low-rank bf16-gradient blocks with random sizes (mostly multiples of 8, rows of whole vectors; otherwise any
    size, which the stripe products finish behind their loops), ranks on and between the class and vector boundaries, every
    kind of second moment."""
    blocks = []
    for b in range(rng.randint(2, 4)):
        if rng.random() < 0.7:
            m, n = 8 * rng.randint(2, 90), 8 * rng.randint(2, 90)
        else:
            m, n = rng.randint(9, 500), rng.randint(9, 500)
        r = min(rng.choice([1, 3, 4, 7, 8, 16, 20, 31, 32, 33, 48, 51, 64, 65, 80, 100, 127, 128]), m, n)
        vm = rng.choice(["element", "rowgroup", "rowgroup", "whole"])
        g = rng.choice([d for d in (1, 2, 3, 4, 5, 8, 16, 32, 64, 128) if m % d == 0]) if vm == "rowgroup" else 1
        pd = rng.choice(["bf16", "bf16", "f32"])
        blocks.append(BlockSpec(f"c{case}b{b}_{m}x{n}_r{r}_{vm}{g}_{pd}", m, n, pd, "bf16", "lowrank", r, vm, g, 1.0,
                                rng.choice([0.0, 0.1])))
    return WL.Workload(f"random{case}", tuple(blocks), steps=5, seed=100 + case, signal_rank=24)


@pytest.mark.parametrize("seed", [2, 3])
def test_random_tables_on_the_mfma_path(seed):
    import random
    rng = random.Random(seed)
    for case in range(10):
        wl = random_table(rng, case)
        hp = dict(T=rng.choice([1, 1, 2, 3]), K=rng.choice([2, 3, 5, 5]), contraction=B.ADAPM_CONTRACT_BF16X2)
        if rng.random() < 0.25:
            hp["normalise"] = 1
        if rng.random() < 0.2:
            hp["bias_correction"] = 0
        clip = rng.choice([None, None, 0.5])
        print([b.name for b in wl.blocks], hp, clip, flush=True)
        run(wl, 5, hp, tol_state=TOL16, tol_param=TOL16, grad_clip=clip)


def test_random_tables_of_every_regime_on_the_exact_path():
    """Random sizes (vectors included), regimes, dtypes, second-moment kinds and flags at the fp32 tolerance."""
    import random
    rng = random.Random(1)
    for case in range(12):
        blocks = []
        for b in range(rng.randint(2, 5)):
            mom = rng.choice(["none", "full", "full", "lowrank", "lowrank"])
            m, n = (rng.randint(1, 3000), 1) if rng.random() < 0.2 else (rng.randint(1, 400), rng.randint(1, 400))
            if mom == "lowrank" and (m < 2 or n < 2):
                mom = "full"
            r = max(1, min(rng.choice([1, 2, 5, 8, 16, 33, 64]), m, n)) if mom == "lowrank" else 0
            vm = rng.choice(["element", "rowgroup", "rowgroup", "whole"])
            g = rng.choice([d for d in (1, 2, 3, 4, 5, 7, 8, 16, 25, 32, 64, 100, 128) if m % d == 0]) if vm == "rowgroup" else 1
            pd, gd = rng.choice(["bf16", "f32"]), rng.choice(["bf16", "f32"])
            blocks.append(BlockSpec(f"c{case}b{b}_{mom}_{m}x{n}_r{r}_{vm}{g}_{pd}{gd}", m, n, pd, gd, mom, r, vm, g,
                                    0.75 if mom == "none" else 1.0, rng.choice([0.0, 0.1])))
        hp = dict(T=rng.choice([1, 1, 2, 3]), K=rng.choice([1, 2, 3, 5, 5]), contraction=B.ADAPM_CONTRACT_F64)
        if rng.random() < 0.25:
            hp["normalise"] = 1
        if rng.random() < 0.2:
            hp["bias_correction"] = 0
        if rng.random() < 0.2:
            hp.update(adam_debias=1, clip=float("inf"))
        clip = rng.choice([None, None, 0.5])
        wl = WL.Workload(f"random_exact{case}", tuple(blocks), steps=5, seed=200 + case, signal_rank=24)
        print([b.name for b in wl.blocks], hp, clip, flush=True)
        run(wl, 5, hp, tol_state=TOL32, tol_param=TOL32, grad_clip=clip)


@pytest.mark.parametrize("shape,mini", [("gpt2_1p5b", False), ("gpt2_1p5b", True), ("llama_350m", False), ("llama_350m", True)])
def test_paper_partition_layer(shape, mini):
    """One layer (plus an embedding-like block) of the paper's own partition (Sec. 4.1): no momentum at
    0.75 x lr, full momentum, low-rank momentum with r = 5 % (80 resp. 51: between the rank classes)."""
    full = WL.paper_partition(shape, mini)
    names = [b.name for b in full.blocks if b.name.startswith("h0.")]
    if shape == "gpt2_1p5b":
        names = ["wpe"] + names
    run(WL.subset(full, names), 5, dict(T=3), tol_state=TOL16, tol_param=TOL16, check_every=2)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_global_gradient_clipping_on_the_exact_path(hp):
    """Sec. 5.1 set-ups: global gradient-norm clipping folded into the step (every regime, every kind of v)."""
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_F64)
    pair, _ = run(mixed_table(), 6, hp, tol_state=TOL32, tol_param=TOL32, check_every=2, grad_clip=1.0)
    assert pair.opt.last_grad_norm()[1] < 1.0              # the clipping was active


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3), dict(T=2, bias_correction=0)])
def test_global_gradient_clipping_on_the_mfma_path(hp):
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2)
    pair, _ = run(ragged_bf16_table(), 6, hp, tol_state=TOL16, tol_param=TOL16, check_every=2, grad_clip=0.5)
    assert pair.opt.last_grad_norm()[1] < 1.0
    run(odd_rank_table(), 4, hp, tol_state=TOL16, tol_param=TOL16, check_every=2, grad_clip=0.5)


def test_global_gradient_clipping_above_the_norm_changes_nothing():
    wl = ragged_bf16_table()
    a, _ = run(wl, 3, dict(T=2, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOL16, tol_param=TOL16, grad_clip=1e9)
    b, _ = run(wl, 3, dict(T=2, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOL16, tol_param=TOL16)
    assert a.opt.last_grad_norm()[1] == 1.0
    for x, y in zip(a.params, b.params):
        assert torch.equal(x, y)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_scale_normalised_alg2_on_the_exact_path(hp):
    """The optional normalised step sizes of Alg. 2 (beyond the paper), every regime, also at a gradient scale where
    the printed iteration overflows."""
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_F64, normalise=1)
    run(mixed_table(), 6, hp, tol_state=TOL32, tol_param=TOL32, check_every=2)
    run(mixed_table(), 4, hp, tol_state=TOL32, tol_param=TOL32, check_every=2, grad_scale=40.0)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3), dict(T=2, bias_correction=0)])
def test_scale_normalised_alg2_on_the_mfma_path(hp):
    hp = dict(hp, contraction=B.ADAPM_CONTRACT_BF16X2, normalise=1)
    run(ragged_bf16_table(), 6, hp, tol_state=TOL16, tol_param=TOL16, check_every=2)
    run(odd_rank_table(), 4, hp, tol_state=TOL16, tol_param=TOL16, check_every=2, grad_scale=0.01)


def test_literal_zero_start_stays_zero_on_gpu():
    wl = WL.subset(WL.tiny_block(), ["attn.q"])
    pair, _ = run(wl, 3, dict(seed=0))
    sv = pair.opt.state_view(0)
    assert float(sv["L"].abs().max()) == 0.0 and float(sv["R"].abs().max()) == 0.0


# ---------------------------------------------------------------------------------------------------------------
# The five configurations at their own step counts.  Blocks are independent in the method, so where the oracle would
# need too long for a whole table it follows a stratified subset at full size: one block of every distinct
# (shape, momentum regime, kind of second moment).  Embedding-sized full-momentum blocks (tens of millions of
# elements, seconds per oracle step) are followed for a few steps only: their update is a linear recursion per
# element with no iteration whose error could grow.
# ---------------------------------------------------------------------------------------------------------------
def f32_params(wl):
    """The same workload with fp32 parameters (bf16 gradients kept): on the MFMA path this shows the arithmetic
    itself, without the bf16 rounding of W."""
    return dataclasses.replace(wl, blocks=tuple(dataclasses.replace(b, param_dtype="f32") for b in wl.blocks))


def test_config2_llama60m_whole_table():
    """All 74 blocks (embedding with full momentum, 56 low-rank matrices at r = 32, 17 norm vectors)."""
    run(WL.llama_60m(), 10, dict(T=1), check_every=5)


def test_config2_llama60m_layer_100_steps():
    full = WL.llama_60m()
    names = [b.name for b in full.blocks if b.name.startswith("l0.")] + ["norm_f"]
    run(WL.subset(full, names), 100, dict(T=1), check_every=10)


def test_config2_llama60m_layer_100_steps_R_held():
    full = WL.llama_60m()
    run(WL.subset(full, ["l0.attn.q", "l0.ffn.gate", "l0.ffn.down", "l0.norm1"]), 100, dict(T=10), check_every=10)


C3_STRATA = ["wpe", "h3.attn.q", "h3.mlp.fc", "h3.mlp.proj", "h3.ln1"]


def test_config3_gpt2_350m_strata_100_steps():
    run(WL.subset(WL.gpt2_350m(), C3_STRATA), 100, dict(T=1), tol_state=TOLX_LONG, tol_param=TOLX_LONG, check_every=10)


def test_config3_gpt2_350m_strata_100_steps_R_held():
    run(WL.subset(WL.gpt2_350m(), ["h3.attn.q", "h3.mlp.proj", "h3.ln1"]), 100, dict(T=100), tol_state=TOLX_LONG,
        tol_param=TOLX_LONG, check_every=10)


def test_config3_strata_100_steps_on_the_exact_path():
    """The same bf16-parameter strata with the fp64 contractions: state at the fp32 tolerance after 100 steps,
    parameters by the bf16 criterion."""
    run(WL.subset(WL.gpt2_350m(), ["h3.attn.q", "h3.mlp.proj", "h3.ln1"]), 100, dict(T=1, contraction=B.ADAPM_CONTRACT_F64),
        tol_state=TOL32, tol_param=TOL32, check_every=20)


def test_config3_gpt2_350m_embedding():
    run(WL.subset(WL.gpt2_350m(), ["wte"]), 3, dict(T=1), tol_state=TOLX, tol_param=TOLX)


def test_config3_strata_with_fp32_parameters_on_the_mfma_path():
    """The arithmetic of the MFMA path without the bf16 rounding of W: parameters, state and product L R of the
    warm-started iteration against the oracle after 100 steps."""
    wl = f32_params(WL.subset(WL.gpt2_350m(), ["h3.attn.q", "h3.mlp.proj"]))
    run(wl, 100, dict(T=1, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOLX_LONG, tol_param=TOLX_LONG, check_every=10)


def test_config4_llama1b_strata_50_steps():
    """2048 x 2048 and 2048 x 5461 (rows of G at 2-byte alignment), per-head gradient scales over two decades."""
    run(WL.subset(WL.llama_1b(), ["l5.attn.k", "l5.ffn.down", "l5.norm1"]), 50, dict(T=1), tol_state=TOLX_LONG,
        tol_param=TOLX_LONG, check_every=10)


def test_config4_llama1b_odd_row_count():
    """5461 x 2048: the last stripes of rows and of columns of G are ragged."""
    run(WL.subset(WL.llama_1b(), ["l5.ffn.gate"]), 10, dict(T=1), tol_state=TOLX_LONG, tol_param=TOLX_LONG)


def test_config4_llama1b_strata_R_held():
    run(WL.subset(WL.llama_1b(), ["l5.attn.k"]), 50, dict(T=100), tol_state=TOLX_LONG, tol_param=TOLX_LONG, check_every=10)
    run(WL.subset(WL.llama_1b(), ["l5.ffn.down", "l5.ffn.gate"]), 6, dict(T=100), tol_state=TOLX_LONG, tol_param=TOLX_LONG)


def test_config4_llama1b_output_head():
    run(WL.subset(WL.llama_1b(), ["lm_head"]), 2, dict(T=1), tol_state=TOLX, tol_param=TOLX)      # embed: same shape and regime


def test_config4_strata_with_fp32_parameters_on_the_mfma_path():
    wl = f32_params(WL.subset(WL.llama_1b(), ["l5.attn.k", "l5.ffn.down"]))
    run(wl, 10, dict(T=1, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOLX_LONG, tol_param=TOLX_LONG, check_every=5)


C5_STRATA = ["h7.attn.q", "h7.attn.v", "h7.mlp.fc", "h7.mlp.proj", "h7.ln1", "wpe"]


@pytest.mark.parametrize("T", [1, 100])
def test_config5_gpt2_1p5b_strata_20_steps(T):
    """Per-head v (Q), per-row v (V, MLP), one v per norm vector, per-row v with full momentum (positions)."""
    run(WL.subset(WL.gpt2_1p5b(), C5_STRATA), 20, dict(T=T), tol_state=TOLX, tol_param=TOLX, check_every=10)


def test_config5_gpt2_1p5b_output_head():
    run(WL.subset(WL.gpt2_1p5b(), ["lm_head"]), 2, dict(T=1), tol_state=TOLX, tol_param=TOLX)


def test_config5_strata_with_fp32_parameters_on_the_mfma_path():
    wl = f32_params(WL.subset(WL.gpt2_1p5b(), ["h7.attn.q", "h7.mlp.fc", "h7.mlp.proj"]))
    run(wl, 20, dict(T=1, contraction=B.ADAPM_CONTRACT_BF16X2), tol_state=TOLX, tol_param=TOLX, check_every=10)


@pytest.mark.parametrize("T", [1, 100])
def test_config5_full_size_sampled_blocks(T):
    """All 388 blocks in the launch configurations the benchmark times (T = 100: one step that runs Alg. 2, then R
    held; T = 1: Alg. 2 every step, the whole-model work lists of its stripe, Gram and update launches); the oracle
    follows a sample of blocks (blocks are independent), the rest is checked for sanity."""
    wl = WL.gpt2_1p5b()
    names = [b.name for b in wl.blocks]
    sample = [names.index(n) for n in ("h0.attn.q", "h23.attn.o", "h47.mlp.fc", "h11.mlp.proj", "h30.ln2", "ln_f",
                                       "wpe")]
    pair = Pair(wl, dict(T=T))
    w0 = pair.params[names.index("h40.attn.k")].clone()
    for t in range(1, 4):
        pair.step(oracle_only=sample)
    rep = pair.compare(TOLX, TOLX, only=sample)
    print(f"gpt2_1p5b full size, T={T}, sampled blocks:", rep, flush=True)
    torch.cuda.synchronize()
    for i, p in enumerate(pair.params):
        assert bool(torch.isfinite(p.float()).all()), names[i]
    assert bool(torch.isfinite(pair.opt.state.view(torch.float32)).all())
    # blocks the oracle did not follow did move
    assert not torch.equal(pair.params[names.index("h40.attn.k")], w0)


def test_held_R_kernel_that_reads_G_once(monkeypatch):
    """ADAPM_PROJ_KEEP=1: blocks of rank class 128 with bf16 parameters, a blockwise v and at most 1600 columns take
    the step with R held in 64-row stripes whose gradient stays in registers between the two passes.  Same parity bar
    as the two-read kernel; ragged rows, short last chunks, a rank between the classes, v groups inside and beyond
    the stripe."""
    monkeypatch.setenv("ADAPM_PROJ_KEEP", "1")
    mk = BlockSpec
    wl = WL.Workload("keep", (
        mk("heads64", 1600, 1600, "bf16", "bf16", "lowrank", 128, "rowgroup", 64, 1.0, 0.1, 64),
        mk("rows130_cols264_g65", 130, 264, "bf16", "bf16", "lowrank", 128, "rowgroup", 65, 1.0, 0.1),
        mk("r100_g16", 208, 136, "bf16", "bf16", "lowrank", 100, "rowgroup", 16, 1.0, 0.1),
        mk("r80_whole", 96, 1600, "bf16", "bf16", "lowrank", 80, "whole", 1, 1.0, 0.0),
        mk("wide_two_read", 136, 1608, "bf16", "bf16", "lowrank", 128, "rowgroup", 1, 1.0, 0.1),
    ), steps=6, seed=21, signal_rank=40)
    pair = Pair(wl, dict(T=3, contraction=B.ADAPM_CONTRACT_BF16X2))
    for t in range(1, 7):
        if t == 3:
            B.adapm_profile_enable(pair.opt.ctx, True)
        pair.step()
        if t == 3:
            torch.cuda.synchronize()
            labels = set(B.adapm_profile_read(pair.opt.ctx))
            B.adapm_profile_enable(pair.opt.ctx, False)
            assert {"fused_project_keep_r128", "fused_project_r128"} <= labels, labels
    rep = pair.compare(TOLX, TOLX)
    print("held-R kernel that keeps G on chip:", rep, flush=True)
    run(WL.subset(WL.gpt2_1p5b(), ["h7.attn.q", "h7.mlp.fc"]), 4, dict(T=100), tol_state=TOLX, tol_param=TOLX)


def test_rank_deficient_R_passes_the_orthonormalisation_unchanged():
    """T > 1 with factors that are exactly zero (a restored state whose R = 0): R R^T has no Cholesky factor, the
    library leaves such a block's (L, R) as Alg. 2 left them instead of writing NaN, and the steps then equal the
    literal zero start of Alg. 1 (factors stay 0, m^c = G), which the oracle computes with seed = 0, T = 1."""
    for names, wl0 in ((["attn.q"], WL.tiny_block()), (["h0.attn.q"], WL.gpt2_350m())):
        wl = WL.subset(wl0, names)
        pair = Pair(wl, dict(T=2))
        pair.opt.state_view(0)["R"].zero_()
        B.adapm_state_loaded(pair.opt.ctx)
        hp_o = O.HParams(beta1=wl.beta1, beta2=wl.beta2, eps=wl.eps, clip=wl.clip, K=wl.K, T=1, seed=0)
        st_o = O.init_state(pair.blocks_o, hp_o)
        W_o = pair.W_o
        for t in range(1, 4):
            grads = pair.stream.next()
            pair.opt.step(pair.params, grads, t, wl.lr)
            W_o, st_o = O.step(pair.blocks_o, hp_o, W_o, [to_np(g) for g in grads], st_o, t, wl.lr)
        torch.cuda.synchronize()
        sv = pair.opt.state_view(0)
        assert float(sv["L"].abs().max()) == 0.0 and float(sv["R"].abs().max()) == 0.0
        assert bool(torch.isfinite(pair.params[0].float()).all())
        pair.W_o, pair.state_o, pair.t = W_o, st_o, 3
        pair.compare(TOLX, TOL32 if wl.blocks[0].param_dtype == "f32" else TOLX)


def test_two_runs_are_bit_identical_and_resume_from_a_state_copy():
    wl = mixed_table()
    hp = dict(T=2)

    def go(nsteps, resume_at=None):
        pair = Pair(wl, hp)
        saved = None
        for t in range(1, nsteps + 1):
            if resume_at is not None and t == resume_at + 1:
                # checkpoint = the flat state buffer (+ step count): restore into a fresh optimizer
                from paper_2510_09103_amd.optimizer import AdaPM
                fresh = AdaPM(wl.blocks, pair.hp_c)
                fresh.state.copy_(saved)
                B.adapm_state_loaded(fresh.ctx)
                pair.opt = fresh
            grads = pair.stream.next()
            pair.t = t
            pair.opt.step(pair.params, grads, t, wl.lr)
            if resume_at is not None and t == resume_at:
                torch.cuda.synchronize()
                saved = pair.opt.state.clone()
        torch.cuda.synchronize()
        return [p.clone() for p in pair.params], pair.opt.state.clone()

    p1, s1 = go(6)
    p2, s2 = go(6)
    p3, s3 = go(6, resume_at=3)
    for a, b, c in zip(p1, p2, p3):
        assert torch.equal(a, b) and torch.equal(a, c)
    assert torch.equal(s1, s2) and torch.equal(s1, s3)


def test_restoring_a_state_into_a_live_optimizer():
    """bf16 blocks on the MFMA path keep derived copies of R between refreshes: after the caller
    overwrites the state buffer, adapm_state_loaded() must make the next step rebuild them."""
    wl = WL.subset(WL.gpt2_350m(), ["h0.attn.q", "h0.mlp.fc"])
    hp = dict(T=4)
    a = Pair(wl, hp)
    for _ in range(6):
        a.step()                                  # t = 5 refreshed; the copies of R belong to that refresh
    torch.cuda.synchronize()
    b = Pair(wl, hp)
    for _ in range(2):
        b.step()                                  # t = 1 refreshed
    torch.cuda.synchronize()
    saved_state, saved_params = b.opt.state.clone(), [p.clone() for p in b.params]
    # continue b to t = 3 for the expected result
    g3 = b.step()
    torch.cuda.synchronize()
    want = [p.clone() for p in b.params]
    # restore b's t = 2 checkpoint into optimizer a (same workspace as its last refresh) and redo t = 3
    a.opt.state.copy_(saved_state)
    B.adapm_state_loaded(a.opt.ctx)
    a.opt.step(saved_params, g3, 3, wl.lr)
    torch.cuda.synchronize()
    for x, y in zip(saved_params, want):
        assert torch.equal(x, y)


@pytest.mark.parametrize("hp", [dict(T=1), dict(T=3)])
def test_degenerate_inputs_zero_gradients_and_zero_step_size(hp):
    """Two degenerate inputs on both contraction paths.  (i) Gradients that are exactly zero from the first step
    on: v stays 0, every momentum stays 0, only the decoupled decay moves W.  (ii) lr = 0: the state advances,
    the parameters must not change by a single bit."""
    wl = WL.Workload("degenerate", ragged_bf16_table().blocks[:3] + WL.subset(WL.tiny_block(), ["attn.q", "norm1"]).blocks,
                     steps=4, seed=3, signal_rank=16)
    pair, _ = run(wl, 4, hp, tol_state=TOL16, tol_param=TOL16, grad_scale=0.0)
    for i in range(len(wl.blocks)):
        sv = pair.opt.state_view(i)
        assert float(sv["v"].abs().max()) == 0.0
        if "L" in sv:
            assert float(sv["L"].abs().max()) == 0.0
    frozen = Pair(wl, hp)
    before = [p.clone() for p in frozen.params]
    for _ in range(3):
        frozen.step(lr=0.0)
    torch.cuda.synchronize()
    for a, b in zip(before, frozen.params):
        assert torch.equal(a, b)
    frozen.compare(TOL16, TOL16)


@pytest.mark.parametrize("rows,cols", [(136, 1 << 21), (1 << 21, 136)])
def test_largest_blocks_of_the_mfma_path_agree_with_the_exact_path(rows, cols):
    """Maximum sizes: 2^21 columns is the widest block the MFMA kernels take (32-bit offsets inside a stripe),
    2^21 rows a tall one whose transposed product still runs in stripes.  The oracle needs minutes at these sizes, so the
    property checked is that the two contraction paths of the library, which share no kernel for low-rank blocks, agree on
    the same inputs."""
    paths_agree(rows, cols, "rowgroup")


@pytest.mark.parametrize("rows,cols", [(200, (1 << 21) - 1), (1 << 21, 137)])
def test_largest_ragged_blocks_agree_with_the_exact_path(rows, cols):
    """The same for rows that are no whole vectors, with a per-element second moment (whose state is what leaves room for
    the stripes' images): the largest offsets of the loads at 2-byte alignment and of the 16-byte second moments."""
    assert "alg2_stripe_step_r32" in paths_agree(rows, cols, "element")


def paths_agree(rows, cols, v_mode):
    from paper_2510_09103_amd.optimizer import AdaPM, make_hparams
    wl = WL.Workload("largest", (BlockSpec("big", rows, cols, "bf16", "bf16", "lowrank", 32, v_mode, 1, 1.0, 0.1),),
                     steps=3, seed=11, signal_rank=8)
    stream = WL.GradientStream(wl, device="cuda:0")
    grads = [[g.clone() for g in stream.next()] for _ in range(3)]
    out = []
    for mode in (B.ADAPM_CONTRACT_BF16X2, B.ADAPM_CONTRACT_F64):
        hp = make_hparams(beta1=wl.beta1, beta2=wl.beta2, eps=wl.eps, clip=wl.clip, K=wl.K, T=2, contraction=mode)
        opt = AdaPM(wl.blocks, hp)
        assert B.adapm_block_contraction(opt.ctx, 0) == mode
        params = WL.initial_params(wl, device="cuda:0")
        for t in range(1, 4):
            opt.step(params, grads[t - 1], t, wl.lr)
        torch.cuda.synchronize()
        sv = opt.state_view(0)
        out.append((params[0].float().clone(), (sv["L"].double()[:4096] @ sv["R"].double()[:, :4096]).clone(), sv["v"].clone()))
        if mode == B.ADAPM_CONTRACT_BF16X2:
            labels = labels_of_a_step(opt, params, grads[0], 1, wl.lr)
        opt.close()
        del opt
    (w_a, lr_a, v_a), (w_b, lr_b, v_b) = out
    scale = float(w_b.abs().mean())
    assert float((w_a - w_b).abs().max()) <= 2 * 2.0 ** -8 * max(float(w_b.abs().max()), scale)     # two bf16 ulps
    assert float((w_a != w_b).float().mean()) < 5e-3
    rms = float(lr_b.pow(2).mean().sqrt())
    assert float((lr_a - lr_b).abs().max()) <= TOL16 * max(float(lr_b.abs().max()), rms)
    assert torch.allclose(v_a, v_b, rtol=1e-5, atol=0.0)
    return labels


def test_one_context_serving_two_state_buffers():
    """The derived copies of R in the workspace belong to one state buffer: a context that steps two replicas
    (two state buffers, one workspace) in turn must rebuild them whenever the state buffer changes."""
    from paper_2510_09103_amd.optimizer import AdaPM, make_hparams
    wl = WL.subset(WL.gpt2_350m(), ["h0.attn.q", "h0.mlp.fc"])
    hp = make_hparams(beta1=wl.beta1, beta2=wl.beta2, eps=wl.eps, clip=wl.clip, K=wl.K, T=4)
    stream = WL.GradientStream(wl, device="cuda:0")
    grads = [[g.clone() for g in stream.next()] for _ in range(6)]
    seqs = [grads, grads[::-1]]                      # the two replicas see different gradients
    want = []
    for k in (0, 1):                                 # each replica with a context of its own
        opt = AdaPM(wl.blocks, hp)
        params = WL.initial_params(wl, device="cuda:0")
        for t in range(1, 7):
            opt.step(params, seqs[k][t - 1], t, wl.lr)
        torch.cuda.synchronize()
        want.append((params, opt.state.clone()))
    shared = AdaPM(wl.blocks, hp)
    states = [shared.state, shared.state.clone()]    # the seeded start is the same for both
    params = [WL.initial_params(wl, device="cuda:0"), WL.initial_params(wl, device="cuda:0")]
    for t in range(1, 7):
        for k in (0, 1):
            shared.state = states[k]
            shared.step(params[k], seqs[k][t - 1], t, wl.lr)
    torch.cuda.synchronize()
    for k in (0, 1):
        for x, y in zip(params[k], want[k][0]):
            assert torch.equal(x, y), f"replica {k}"
        assert torch.equal(states[k], want[k][1]), f"replica {k}"


def test_step_rejects_bad_arguments_on_device():
    wl = WL.subset(WL.tiny_block(), ["norm1"])
    pair = Pair(wl)
    g = pair.stream.next()
    with pytest.raises(B.AdapmError) as e:
        pair.opt.step(pair.params, g, 0, 1e-3)
    assert e.value.status == B.ADAPM_ESTATE
    w_before = pair.params[0].clone()
    pair.opt.step(pair.params, g, 1, 1e-3)
    torch.cuda.synchronize()
    assert not torch.equal(w_before, pair.params[0])
