"""Work lists that the planner makes, read out of a context on the host: no GPU."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2510_09103_amd import binding as B
from paper_2510_09103_amd.build import CSRC, FLAGS
from paper_2510_09103_amd.optimizer import make_hparams

PROBE = r'''
#include "adapm_api.hip"
// One row of `out` per workgroup of launch `op` of a step: problem (-1: padding), ti, tj, nj, M, N, tile height, tile width, length of
// the contractions.  Returns the number of rows, -1 past the last launch, 0 for launches that are no tiles of the exact path.
extern "C" int64_t probe_tiles(const adapm_ctx* c, int held, int64_t op, const char** label, int64_t* out, int64_t cap) {
  const std::vector<Op>& seq = held ? c->seq_project : c->seq_refresh;
  if (op >= (int64_t)seq.size()) return -1;
  *label = seq[op].label;
  if (seq[op].kind != OP_GEMM && seq[op].kind != OP_UPDATE64) return 0;
  const GemmList& gl = c->gemms[seq[op].index];
  if ((int64_t)gl.tiles.size() > cap) return -2;
  for (const GemmTile& t : gl.tiles) {
    if (t.prob == GEMM_TILE_NONE) { *out = -1; out += 9; continue; }
    const GemmProblem& p = gl.probs[t.prob];
    const int64_t row[9] = {t.prob, t.ti, t.tj, t.nj, p.M, p.N, 16 * p.tm, 16 * p.tn, (int64_t)p.K1 + p.K2 + p.K3};
    for (int64_t x : row) *out++ = x;
  }
  return (int64_t)gl.tiles.size();
}
'''


# Waves of a workgroup of launch `op` (plus 100 where they request operands a step ahead), 0 for launches of another kind, -1 past the last one
PROBE += r'''
// groups of the workgroup `i` of the grouped update, -1 past the last one
extern "C" int64_t probe_groups(const adapm_ctx* c, int64_t i) { return i < (int64_t)c->grp.h.size() ? c->grp.h[i].ngroups : -1; }
// is block i's gradient read non-temporally by the update of blocks without low-rank momentum?
extern "C" int64_t probe_last_read(const adapm_ctx* c, int64_t i) { return c->blocks.h[i].g_last; }
extern "C" int64_t probe_launch(const adapm_ctx* c, int held, int64_t op, const char** label) {
  const std::vector<Op>& seq = held ? c->seq_project : c->seq_refresh;
  if (op >= (int64_t)seq.size()) return -1;
  *label = seq[op].label;
  return seq[op].kind == OP_GEMM ? c->gemms[seq[op].index].waves + 100 * c->gemms[seq[op].index].ahead : 0;
}
'''


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("probe")
    (d / "probe.hip").write_text(PROBE)
    lib = d / "libprobe.so"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *FLAGS, "-O1", "-shared", "-I", CSRC, str(d / "probe.hip"), "-o", str(lib),
                    "-L" + os.path.dirname(B.LIB_PATH), "-l:" + os.path.basename(B.LIB_PATH), "-Wl,-rpath," + os.path.dirname(B.LIB_PATH)], check=True, stderr=subprocess.DEVNULL)
    return C.CDLL(str(lib))


class Plan:
    def __init__(self, lib, table, hp):
        self.lib, self.ctx = lib, C.c_void_p()
        arr = (B.adapm_block_t * len(table))(*table)
        assert lib.adapm_init(C.byref(self.ctx), arr, C.c_int64(len(table)), C.byref(hp)) == B.ADAPM_OK

    def __enter__(self):
        return self

    def __exit__(self, *_):
        self.lib.adapm_destroy(self.ctx)

    def launches(self, held):
        """(label, rows of probe_tiles) of the step's launches of tiles"""
        self.lib.probe_tiles.restype = C.c_int64
        cap = 200000
        out, label = (C.c_int64 * (9 * cap))(), C.c_char_p()
        op = 0
        while True:
            n = self.lib.probe_tiles(self.ctx, C.c_int(held), C.c_int64(op), C.byref(label), out, C.c_int64(cap))
            assert n != -2
            if n < 0:
                return
            if n > 0:
                yield label.value.decode(), [tuple(out[9 * i:9 * i + 9]) for i in range(n)]
            op += 1


    def labels(self, held):
        """(label, what probe_launch says of it) of every launch of a step"""
        self.lib.probe_launch.restype = C.c_int64
        label, op = C.c_char_p(), 0
        while (w := self.lib.probe_launch(self.ctx, C.c_int(held), C.c_int64(op), C.byref(label))) >= 0:
            yield label.value.decode(), w
            op += 1

    def waves(self, held):
        out = {}
        for label, w in self.labels(held):
            if w > 0:
                out.setdefault(label, set()).add(w)
        return out


DT = {"f32": B.ADAPM_F32, "bf16": B.ADAPM_BF16}


def lowrank(m, n, r, pd="f32", gd="bf16", v=B.ADAPM_V_ELEMENT):
    return B.adapm_block_t(rows=m, cols=n, param_dtype=DT[pd], grad_dtype=DT[gd], mom_mode=B.ADAPM_MOM_LOWRANK, rank=r, v_mode=v,
                           v_group_rows=1, lr_scale=1.0, weight_decay=0.1)


def layers(d, f, r, count, up=1, attention=4):
    return count * ([lowrank(d, d, r)] * attention + [lowrank(f, d, r)] * up + [lowrank(d, f, r)])


FEW = {
    "one": [lowrank(4096, 4096, 128)],
    "two": 2 * [lowrank(4096, 4096, 128)],
    "three_unlike": [lowrank(4096, 1024, 64), lowrank(512, 512, 64), lowrank(1000, 3001, 100)],
    "layer_2048": layers(2048, 8192, 128, 1),
    "layer_2048_two_lowrank": layers(2048, 8192, 128, 1, attention=2),
    "layer_1024_gated": layers(1024, 2731, 64, 1, up=2),
    "layer_512_gated": layers(512, 1376, 32, 1, up=2),
    "two_layers_1024": layers(1024, 4096, 64, 2),
    "fourteen": layers(1024, 2731, 64, 2, up=2),
    "eight_layers_512": layers(512, 1376, 32, 8, up=2),
}


@pytest.mark.parametrize("T", [1, 10])
@pytest.mark.parametrize("name", FEW)
def test_tiles_of_the_exact_path_fill_the_xcds_evenly(probe, name, T):
    """Workgroup i runs on XCD i mod 8.  A launch that fills the chip puts no more than 1.15 times the mean of its multiply-adds on any
    XCD, and every tile of every result is there exactly once."""
    seen = 0
    with Plan(probe, FEW[name], make_hparams(T=T)) as plan:
        for held in range(2 if T > 1 else 1):
            for label, rows in plan.launches(held):
                load, covered, shape = [0.0] * 8, {}, {}
                for i, (prob, ti, tj, nj, M, N, th, tw, K) in enumerate(rows):
                    if prob < 0:
                        continue
                    load[i % 8] += K * nj
                    shape[prob] = (-(-M // th), -(-N // tw))
                    covered.setdefault(prob, []).extend((ti, tj + k) for k in range(nj))
                for prob, (nti, ntj) in shape.items():
                    want = {(a, b) for a in range(nti) for b in range(ntj)}
                    got = covered[prob]
                    assert len(got) == len(set(got)), label
                    assert set(got) == want or (label == "regauge_gram_f64" and set(got) == {(a, b) for a, b in want if b <= a}), label
                if sum(r[0] >= 0 for r in rows) >= 768:
                    seen += 1
                    assert max(load) * 8 <= 1.15 * sum(load), (label, len(rows), [round(8 * x / sum(load), 2) for x in load])
    assert seen or name in ("layer_512_gated", "three_unlike")


@pytest.mark.parametrize("side,launches", [(256, 1), (1024, 4)])
def test_few_tiles_of_several_types_are_one_update(probe, side, launches):
    """A kernel per type of G, W and second moment costs a launch each: where all of them together are few tiles, one launch takes
    them all."""
    V = (B.ADAPM_V_ELEMENT, B.ADAPM_V_ROWGROUP)
    table = [lowrank(side, side, 8, "f32", gd, v) for gd in ("f32", "bf16") for v in V] * 6
    with Plan(probe, table, make_hparams(T=10)) as plan:
        rows = [r for label, r in plan.launches(1) if label == "update_lowrank_f64"]
    assert len(rows) == launches


@pytest.mark.parametrize("k,m,n,r,update,project", [
    (1, 256, 256, 8, 8, 8), (2, 512, 512, 32, 8, 8), (1, 1024, 1024, 64, 8, 8), (1, 8192, 2048, 8, 8, 4), (16, 128, 128, 8, 8, 8),
    (5, 512, 512, 16, 4, 8), (10, 256, 256, 16, 4, 8), (4, 1024, 1024, 32, 4, 8), (2, 2048, 2048, 16, 4, 8), (16, 256, 256, 32, 4, 8), (36, 128, 128, 16, 4, 8),
    (60, 128, 128, 16, 4, 4), (4, 1024, 1024, 64, 4, 4), (1, 2048, 2048, 128, 4, 4), (100, 64, 64, 8, 4, 8)])
def test_waves_follow_from_how_a_launch_fills_the_chip(probe, k, m, n, r, update, project):
    """Eight waves on small tiles only where a launch leaves compute units idle: every table here was measured both ways."""
    with Plan(probe, [lowrank(m, n, r) for _ in range(k)], make_hparams(T=10)) as plan:
        assert {w % 100 for w in plan.waves(0)["alg2_update_f64"]} == {update}
        assert {w % 100 for w in plan.waves(1)["project_f64"]} == {project}
        assert all(w % 100 in (4, 8) for ws in plan.waves(0).values() for w in ws)


@pytest.mark.parametrize("k,m,n,r,ahead", [(1, 2048, 2048, 128, True), (4, 1024, 1024, 32, True), (1, 4096, 4096, 8, True), (1, 256, 256, 8, True),
                                           (100, 64, 64, 8, False), (6, 512, 512, 128, False), (16, 512, 512, 64, False), (200, 96, 96, 12, False)])
def test_operands_are_requested_ahead_where_a_launch_does_not_fill_the_chip(probe, k, m, n, r, ahead):
    """... and not where it does, where the registers serve a fourth wave better; with R held always."""
    with Plan(probe, [lowrank(m, n, r) for _ in range(k)], make_hparams(T=10)) as plan:
        assert {w > 100 for w in plan.waves(0)["alg2_update_f64"]} == {ahead}
        assert {w > 100 for w in plan.waves(1)["project_f64"]} == {True}


@pytest.mark.parametrize("m,n,r", [(1024, 1024, 64), (512, 2048, 128), (700, 300, 17), (4096, 64, 8), (2048, 2048, 128)])
def test_copies_of_the_factors_do_not_split_a_group(probe, m, n, r):
    """From two GD iterations on the exact path keeps the previous factors in its scratch (K = 5; not with one, K = 2).  Tables of a
    small state, whose scratch has a fixed bound, run in as many groups either way, inside the array of adapm_step_static where
    they did."""
    def plan_of(k, K):
        with Plan(probe, [lowrank(m, n, r, v=B.ADAPM_V_ROWGROUP) for _ in range(k)], make_hparams(T=1, K=K)) as plan:
            probe.adapm_workspace_bytes.restype = probe.adapm_state_bytes.restype = C.c_size_t
            runs = sum(label == "alg2_update_f64" for label, _ in plan.labels(0))
            return runs // (4 if K == 5 else 1), probe.adapm_workspace_bytes(plan.ctx), probe.adapm_state_bytes(plan.ctx)
    seen = set()
    for k in range(1, 400):
        one, ws_one, state = plan_of(k, 2)
        if state > 32 << 20:
            break
        many, ws_many, _ = plan_of(k, 5)
        assert many <= one, k
        assert ws_one > B.adapm_static_scratch_bytes() or ws_many <= B.adapm_static_scratch_bytes(), k
        seen.add(one)
    assert len(seen) > 1


@pytest.mark.parametrize("mom,v,side,last", [
    (B.ADAPM_MOM_FULL, B.ADAPM_V_ELEMENT, 18, 0), (B.ADAPM_MOM_FULL, B.ADAPM_V_ELEMENT, 32, 1), (B.ADAPM_MOM_NONE, B.ADAPM_V_ROWGROUP, 64, 0),
    (B.ADAPM_MOM_NONE, B.ADAPM_V_ROWGROUP, 128, 1), (B.ADAPM_MOM_FULL, B.ADAPM_V_ROWGROUP, 32, 0), (B.ADAPM_MOM_FULL, B.ADAPM_V_ROWGROUP, 48, 1)])
def test_gradients_of_tables_that_stay_in_the_caches_are_not_sent_out_of_them(probe, mom, v, side, last):
    """Blocks of 2^20 elements without low-rank momentum: the non-temporal read of G costs up to a fifth of a step whose gradients, parameters
    and state fit the last-level cache (256 MiB) and pays where they do not."""
    table = [B.adapm_block_t(rows=1024, cols=1024, param_dtype=B.ADAPM_BF16, grad_dtype=B.ADAPM_BF16, mom_mode=mom, rank=0, v_mode=v, v_group_rows=1,
                             lr_scale=1.0, weight_decay=0.1) for _ in range(side)]
    with Plan(probe, table, make_hparams()) as plan:
        probe.probe_last_read.restype = C.c_int64
        assert {probe.probe_last_read(plan.ctx, C.c_int64(i)) for i in range(side)} == {last}


@pytest.mark.parametrize("rows,cols,share", [(1, 64, 1), (3000, 192, 4), (4096, 1024, 4), (4097, 1024, 8), (8192, 1024, 8), (8193, 64, 8), (16384, 512, 8),
                                             (16385, 512, 12), (50257, 1600, 20), (40000, 2048, 16)])
def test_groups_are_spread_over_the_chip(probe, rows, cols, share):
    """One group per wave while all run at once, two of them up to 8192 groups, then between 1024 and 2048 workgroups until one has
    32768 elements."""
    table = [B.adapm_block_t(rows=rows, cols=cols, param_dtype=B.ADAPM_BF16, grad_dtype=B.ADAPM_BF16, mom_mode=B.ADAPM_MOM_FULL, rank=0,
                             v_mode=B.ADAPM_V_ROWGROUP, v_group_rows=1, lr_scale=1.0, weight_decay=0.1)]
    with Plan(probe, table, make_hparams()) as plan:
        probe.probe_groups.restype = C.c_int64
        got, i = [], 0
        while (n := probe.probe_groups(plan.ctx, C.c_int64(i))) >= 0:
            got.append(n)
            i += 1
    assert sum(got) == rows and set(got[:-1]) <= {share} and got[-1] <= share and max(got) == share
    assert len(got) >= min(512, rows // 4)
