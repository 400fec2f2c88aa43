"""Listings of the kernels that use the fp64 matrix instruction, built here for gfx950: no GPU.

The hardware does not interlock a read of a v_mfma_f64_16x16x4 result: for 19 wait states (one per instruction, N + 1 for
s_nop N) it returns the register's old contents.  Two rules hold on every path through every kernel:
  - no instruction but another matrix instruction touches a result register earlier than that (the compiler's part);
  - nothing but copies between registers happens to a result before the kernel's own wait, mfma_f64_results() of
    k_f64_common.h, which leaves the line "; fp64 results" (the source's part)."""
import os
import re
import subprocess

import pytest

from paper_2510_09103_amd.build import CSRC, FLAGS

WAIT_STATES = 19
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
FENCE = "; fp64 results"


def registers(text):
    return {(k, i) for k, lo, hi, one in REG.findall(text) for i in range(int(lo or one), int(hi or one) + 1)}


def kernels(listing):
    """(name, lines) of every function: labels, instructions and the marks of the kernel's own waits"""
    name, lines = None, []
    for line in listing.splitlines():
        start = re.match(r"(_Z\w+):", line)
        if start:
            name, lines = start.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            yield name, lines
            name = None
        elif name and FENCE in line:
            lines.append(FENCE)
        elif name:
            code = line.split(";")[0].strip()
            if code and (not code.startswith(".") or code.startswith(".LBB")):
                lines.append(code)


def blocks_of(lines):
    blocks, at = [[]], {}
    for l in lines:
        if l.endswith(":"):
            if blocks[-1]:
                blocks.append([])
            at[l[:-1]] = len(blocks) - 1
        else:
            blocks[-1].append(l)
            if re.match(r"s_(c?branch|endpgm)", l):
                blocks.append([])
    follow = []
    for i, b in enumerate(blocks):
        last = b[-1] if b else ""
        jump = re.match(r"s_c?branch\S*\s+(\S+)", last)
        f = [at[jump.group(1)]] if jump else []
        if not re.match(r"s_(branch|endpgm)\b", last) and i + 1 < len(blocks):
            f.append(i + 1)
        follow.append(f)
    return blocks, follow


def walk(block, age, open_, faults=None):
    """age: wait states since a matrix instruction wrote a register; open_: registers that hold a result (or a copy of one)
    that has not passed the kernel's own wait"""
    age, open_ = dict(age), set(open_)
    for l in block:
        if l == FENCE:
            open_.clear()
            continue
        op, _, args = l.partition(" ")
        first, _, rest = args.partition(",")
        mfma = op.startswith("v_mfma_f64")
        if (op.startswith("v_") and not op.startswith("v_cmp")) or "_load" in op or op.startswith("ds_read"):
            written, read = registers(first), registers(rest)
        else:
            written, read = set(), registers(args)
        copy = op.startswith(("v_mov_b", "v_accvgpr_"))
        if faults is not None and not mfma:
            if any(age.get(r, WAIT_STATES) < WAIT_STATES for r in read):
                faults.append(("early", l))
            if not copy and read & open_:
                faults.append(("no wait", l))
        passed = int(args) + 1 if op == "s_nop" else 1
        age = {r: n + passed for r, n in age.items() if n + passed < WAIT_STATES and r not in written}
        carries = mfma or (copy and read & open_)
        open_ = open_ | written if carries else open_ - written
        if mfma:
            age.update({r: 0 for r in written})
    return age, open_


def faults_of(lines):
    blocks, follow = blocks_of(lines)
    state = {0: ({}, set())}
    todo = [0]
    while todo:
        i = todo.pop()
        age, open_ = walk(blocks[i], *state[i])
        for j in follow[i]:
            a, o = state.get(j, (None, None))
            if a is None:
                state[j] = (dict(age), set(open_))
                todo.append(j)
                continue
            fresh = {r: n for r, n in age.items() if n < a.get(r, WAIT_STATES)}
            if fresh or not open_ <= o:
                a.update(fresh)
                o |= open_
                todo.append(j)
    faults = []
    for i, (age, open_) in state.items():
        walk(blocks[i], age, open_, faults)
    return faults


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    out = tmp_path_factory.mktemp("listings")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    sources = [f for f in sorted(os.listdir(CSRC)) if f.endswith(".hip") and "k_f64_common.h" in open(os.path.join(CSRC, f)).read()]
    procs = [subprocess.Popen([hipcc, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, f), "-o", str(out / f)],
                              stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL) for f in sources]
    assert [p.wait() for p in procs] == [0] * len(procs)
    return [k for f in sources for k in kernels((out / f).read_text()) if any(l.startswith("v_mfma_f64") for l in k[1])]


def test_results_of_the_fp64_matrix_instruction_are_waited_for(listings):
    assert len(listings) >= 3
    for name, lines in listings:
        assert faults_of(lines) == [], name


def test_a_listing_without_its_waits_is_noticed(listings):
    for name, lines in listings:
        assert ("no wait" in {k for k, _ in faults_of([l for l in lines if l != FENCE])}), name
        assert ("early" in {k for k, _ in faults_of([l for l in lines if not l.startswith("s_nop")])}), name
