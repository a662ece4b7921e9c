"""Static check of the generated gfx950 code (no GPU): loads issued from inline assembly are
invisible to the compiler's wait-count bookkeeping, so nothing may read or write their
destination registers before a wait that covers them, on any path.  The kernels guarantee that
by making those registers operands of the wait; this test compiles the kernels to assembly and
follows every path from every such load through the control-flow graph to confirm it.

The model: vector-memory operations of a wave complete in issue order, and `s_waitcnt vmcnt(N)`
returns when at most N of them are outstanding, so a load is complete once a wait with
N <= (vector-memory instructions issued after it) has been passed.  That rule is applied to the
compiler's own waits.  A wait written by hand (inside inline assembly) is taken to cover every
hand-issued load before it: its count is the kernel author's statement about the instructions
in between (the streaming loop waits with vmcnt(loads of the next tile), and both staging paths
issue exactly that many), which a path-insensitive pass over two complementary branches cannot
re-derive.  What this test does establish is that the registers stay untouched up to that wait.

Matrix instructions written in inline assembly are invisible to it as well: the compiler adds no
wait states around them.  They accumulate in place, so between the MFMAs of one accumulator nothing
else may touch it, and nothing may read or write it until SETTLED wait states after the last one; an
operand that a vector instruction writes needs OPERAND wait states before the MFMA.  Every path is
followed for that too.

A store of more than eight bytes a lane reads its registers while the next instructions issue; a vector
instruction that overwrites them has to stay STORED wait states away.  The compiler keeps them, across the ends of
basic blocks too, except behind a buffer store with its offset in a scalar register, where it keeps none.  Every path
behind every such store of every kernel source is followed, and the scalar form is not used."""
import collections
import os
import re
import subprocess

import pytest

from paper_2603_17435_amd import build as zs_build

VMEM = ("global_load", "global_store", "global_atomic", "scratch_load", "scratch_store", "buffer_load", "buffer_store",
        "flat_load", "flat_store", "flat_atomic")
SATURATED = 64  # vmcnt cannot name more


def registers(operand: str) -> set[int]:
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m.group(1))} if m else set()


def kernels(asm: str):
    """(name, [(text, in_inline_asm)]) per kernel of the translation unit."""
    for km in re.finditer(r"^(_Z\w+):.*$", asm, re.M):
        end = asm.find(".end_amdhsa_kernel", km.end())
        nxt = re.search(r"^_Z\w+:.*$", asm[km.end():], re.M)
        if end < 0 or (nxt and km.end() + nxt.start() < end):
            continue
        ins, inline = [], False
        for line in asm[km.end():end].split("\n"):
            if "#ASMSTART" in line:
                inline = True
            if "#ASMEND" in line:
                inline = False
            text = line.split(";")[0].strip()
            if text and (not text.startswith(".") or re.match(r"\.LBB\d+_\d+:", text)):
                ins.append((text, inline))
        yield km.group(1), ins


SETTLED = 16  # what the kernels wait for; a 16x16x32 BF16 MFMA (four passes) needs less
OPERAND = 2


def successor_function(ins):
    label_at = {t[:-1]: i for i, (t, _) in enumerate(ins) if t.endswith(":")}

    def successors(i):
        t = ins[i][0]
        if t.endswith(":"):
            return [i + 1]
        mn = t.split()[0]
        if mn == "s_endpgm":
            return []
        if mn == "s_branch":
            return [label_at[t.split()[1]]]
        if mn.startswith("s_cbranch"):
            return [label_at[t.split()[1]], i + 1]
        return [i + 1]
    return successors


def operands(text):
    parts = text.split(None, 1)
    return parts[0], [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []


def mfma_hazards(ins):
    """Instructions that break the rules above, {index: (text, registers)}."""
    n, successors = len(ins), successor_function(ins)
    state_in = [None] * n  # (accumulator register -> wait states since its MFMA, vector-written register -> wait states since)
    state_in[0] = ({}, {})
    work = collections.deque([0])
    found = {}
    while work:
        i = work.popleft()
        acc, written = (dict(x) for x in state_in[i])
        text, inline = ins[i]
        if not text.endswith(":"):
            mn, ops = operands(text)
            regs = [registers(o.split()[0]) for o in ops if o]
            if inline and mn.startswith("v_mfma"):
                dst, a, b, c = regs
                bad = (a | b) & acc.keys() | (a | b | c) & written.keys()
                if dst != c:
                    bad |= dst | c
                elif dst & acc.keys() and any(acc.get(r, (0, None))[1] != min(dst) for r in dst):
                    bad |= dst  # overlaps another accumulator
            else:
                bad = set().union(*regs) & acc.keys() if regs else set()
            if bad:
                found.setdefault(i, (text, sorted(bad)))
            wait = int(ops[0], 0) + 1 if mn == "s_nop" else 1
            acc = {r: (k + wait, base) for r, (k, base) in acc.items() if k + wait < SETTLED}
            written = {r: k + wait for r, k in written.items() if k + wait < OPERAND}
            if inline and mn.startswith("v_mfma"):
                acc.update({r: (0, min(dst)) for r in dst})
            elif mn.startswith("v_") and regs:
                written.update({r: 0 for r in regs[0]})
        for s in successors(i):
            if s >= n:
                continue
            old = state_in[s]
            new = (acc, written) if old is None else tuple(
                {r: min(x[r], y[r]) if r in x and r in y else x.get(r, y.get(r)) for r in x.keys() | y.keys()} for x, y in zip((acc, written), old))
            if old is None or new != old:
                state_in[s] = new
                work.append(s)
    return found


def hazards(ins):
    n, successors = len(ins), successor_function(ins)
    state_in = [None] * n  # register -> fewest vector-memory instructions issued since its load, over all paths
    state_in[0] = {}
    work = collections.deque([0])
    found = {}
    while work:
        i = work.popleft()
        cur = dict(state_in[i])
        text, inline = ins[i]
        if not text.endswith(":"):
            mn, ops = operands(text)
            if mn == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", text)
                if m:
                    cur = {} if inline else {r: k for r, k in cur.items() if k < int(m.group(1))}
            else:
                asm_load = inline and mn.startswith("global_load") and "lds" not in mn
                touched = set().union(*(registers(o.split()[0]) for o in ops if o)) if ops else set()
                if not asm_load and touched & cur.keys():
                    found.setdefault(i, (text, sorted(touched & cur.keys())))
                if mn.startswith(VMEM):
                    cur = {r: min(k + 1, SATURATED) for r, k in cur.items()}
                if asm_load:
                    for r in registers(ops[0]):
                        cur[r] = 0
        for s in successors(i):
            if s >= n:
                continue
            old = state_in[s]
            new = dict(cur) if old is None else {r: min(cur.get(r, SATURATED), old.get(r, SATURATED)) for r in cur.keys() | old.keys()}
            if old is None or new != old:
                state_in[s] = new
                work.append(s)
    return found


WIDE_STORE = re.compile(r"(global|buffer|flat|scratch)_store_dwordx[34]")
STORED = 2


def wide_store_hazards(ins):
    """Vector instructions that overwrite the data of a wide store fewer than STORED wait states behind it, on any
    path; and wide buffer stores with a scalar register as offset."""
    successors, found = successor_function(ins), {}
    for i, (text, _) in enumerate(ins):
        mn, ops = operands(text)
        if not WIDE_STORE.match(mn):
            continue
        if mn.startswith("buffer") and re.match(r"(s\d+|m0)\b", ops[3]):
            found[i] = (text, "scalar offset")
        data = registers(ops[0].split()[0] if mn.startswith("buffer") else ops[1].split()[0])
        assert data, text
        todo, fewest = [(k, 0) for k in successors(i)], {}
        while todo:
            k, states = todo.pop()
            if k >= len(ins) or states >= STORED or fewest.get(k, STORED) <= states:
                continue
            fewest[k] = states
            nxt = ins[k][0]
            if not nxt.endswith(":"):  # (a label takes no time)
                m, o = operands(nxt)
                if m.startswith("v_") and o and registers(o[0].split()[0]) & data:
                    found[k] = (text, nxt)
                states += int(o[0], 0) + 1 if m == "s_nop" else 1
            todo += [(s, states) for s in successors(k)]
    return found


@pytest.fixture(scope="module")
def asm_of(tmp_path_factory):
    """The generated code of every kernel source, {file name: text}."""
    out = tmp_path_factory.mktemp("isa")
    texts = {}
    for src in (s for s in zs_build.sources() if s.endswith(".hip")):
        to = out / (os.path.basename(src) + ".s")
        cmd = [zs_build.HIPCC, "-S", "--cuda-device-only", src, "-o", str(to)] + \
              [f for f in zs_build.COMMON if f != "-fPIC"] + zs_build.DEVICE
        subprocess.run(cmd, check=True, capture_output=True)
        texts[os.path.basename(src)] = to.read_text()
    return texts


@pytest.fixture(scope="module")
def kernel_asm(asm_of):
    return asm_of["zs_kernels.hip"]


def test_checker_sees_a_planted_hazard():
    """The checker on hand-made code: a register written while its load is in flight is reported,
    the same code with a covering wait is not, and a wait that leaves the load outstanding does not count."""
    def prog(wait):
        return [("s_nop 0", False), ("global_load_dwordx4 v[4:7], v1, s[2:3]", True), ("global_load_lds_dwordx4 v1, s[4:5]", True)] + \
               ([(wait, False)] if wait else []) + [("v_mov_b32_e32 v5, v0", False), ("s_endpgm", False)]
    assert hazards(prog(None))
    assert hazards(prog("s_waitcnt vmcnt(2)"))
    assert not hazards(prog("s_waitcnt vmcnt(1)"))
    assert not hazards(prog("s_waitcnt vmcnt(0)"))
    # a branch around the wait is a path without it
    branchy = [("global_load_dwordx4 v[4:7], v1, s[2:3]", True), ("s_cbranch_scc1 .LBB0_1", False), ("s_waitcnt vmcnt(0)", True),
               (".LBB0_1:", False), ("v_add_f32_e32 v0, v4, v0", False), ("s_endpgm", False)]
    assert hazards(branchy)


def test_no_register_of_a_hand_issued_load_is_touched_before_its_wait(kernel_asm):
    seen_loads = 0
    for name, ins in kernels(kernel_asm):
        seen_loads += sum(1 for t, inline in ins if inline and t.startswith("global_load") and "lds" not in t.split()[0])
        found = hazards(ins)
        assert not found, f"{name}: {list(found.values())[:4]}"
    assert seen_loads > 0  # the streaming kernels issue their activation fragments by hand


def test_checker_sees_planted_mfma_hazards():
    """The same for matrix instructions, on hand-made code."""
    def mfma(acc, a="v[20:23]", b="v[24:27]", c=None):
        return (f"v_mfma_f32_16x16x32_bf16 {acc}, {a}, {b}, {c or acc}", True)
    nop, end = ("s_nop 15", True), ("s_endpgm", False)
    copy = ("v_mov_b32_e32 v30, v2", False)
    assert not mfma_hazards([mfma("v[0:3]"), mfma("v[4:7]"), mfma("v[0:3]"), nop, copy, end])
    assert mfma_hazards([mfma("v[0:3]"), ("s_nop 3", True), copy, end])                     # read too early
    assert mfma_hazards([mfma("v[0:3]"), ("v_mov_b32_e32 v2, 0", False), nop, end])         # written too early
    assert mfma_hazards([mfma("v[0:3]"), ("ds_read_b128 v[0:3], v40", False), nop, end])
    assert mfma_hazards([mfma("v[0:3]"), mfma("v[2:5]"), nop, end])                         # overlapping accumulators
    assert mfma_hazards([mfma("v[0:3]"), mfma("v[4:7]", a="v[0:3]"), nop, end])             # an accumulator as operand
    assert mfma_hazards([mfma("v[0:3]", c="v[4:7]"), nop, end])                             # not in place
    write = ("v_mov_b32_e32 v21, v40", False)
    assert mfma_hazards([write, mfma("v[0:3]"), nop, end])                                  # operand just written
    assert not mfma_hazards([write, ("s_nop 1", True), mfma("v[0:3]"), nop, end])
    # one path of two without the wait, and a copy at the end of a loop
    assert mfma_hazards([mfma("v[0:3]"), ("s_cbranch_scc1 .LBB0_1", False), nop, (".LBB0_1:", False), copy, end])
    assert mfma_hazards([(".LBB0_1:", False), mfma("v[0:3]"), ("v_mov_b32_e32 v3, v9", False), ("s_cbranch_scc1 .LBB0_1", False), end])


def test_hand_written_mfmas_keep_their_accumulators(kernel_asm):
    kernels_with = 0
    for name, ins in kernels(kernel_asm):
        if any(inline and t.startswith("v_mfma") for t, inline in ins):
            kernels_with += 1
            found = mfma_hazards(ins)
            assert not found, f"{name}: {list(found.values())[:4]}"
    assert kernels_with > 0  # the consumers of the shared-decode kernel


def test_checker_sees_an_overwritten_store():
    store, end = ("buffer_store_dwordx4 v[0:3], v9, s[4:7], 0 offen offset:16 sc1", False), ("s_endpgm", False)
    over, label, other = ("v_mov_b32_e32 v2, 0", False), (".LBB0_1:", False), ("s_add_u32 s0, s0, s1", False)

    def nop(n):
        return (f"s_nop {n}", False)
    assert wide_store_hazards([store, over, end])
    assert wide_store_hazards([store, label, over, end])
    assert wide_store_hazards([("global_store_dwordx4 v[8:9], v[0:3], off", False), label, over, end])
    assert wide_store_hazards([store, nop(0), over, end])
    assert wide_store_hazards([store, other, label, over, end])
    assert not wide_store_hazards([store, nop(1), over, end])
    assert not wide_store_hazards([store, nop(0), label, other, over, end])
    assert not wide_store_hazards([store, ("v_mov_b32_e32 v4, 0", False), ("v_mov_b32_e32 v5, 0", False), over, end])
    assert not wide_store_hazards([("global_store_dwordx2 v[8:9], v[2:3], off", False), over, end])
    # one path of two with the wait states, and a loop that comes back
    branch = ("s_cbranch_scc1 .LBB0_1", False)
    assert wide_store_hazards([store, branch, nop(0), label, over, end])
    assert not wide_store_hazards([store, nop(0), branch, nop(3), label, over, end])
    assert wide_store_hazards([label, over, store, branch, end])
    # the offset in a scalar register
    assert wide_store_hazards([("buffer_store_dwordx4 v[0:3], v9, s[4:7], s2 offen sc1", False), nop(3), end])


def test_no_wide_store_loses_its_data(asm_of):
    stores = {}
    for source, asm in asm_of.items():
        for name, ins in kernels(asm):
            stores[source] = stores.get(source, 0) + sum(1 for t, _ in ins if WIDE_STORE.match(t))
            found = wide_store_hazards(ins)
            assert not found, f"{source}: {name}: {list(found.values())[:4]}"
    assert len(stores) == 3 and all(stores.values())


def test_no_kernel_asks_for_private_memory(asm_of):
    """A private segment that a kernel declares is set up for its launches whether it is used or not, which a library that
    promises not to allocate must not ask for."""
    kernels_seen = 0
    for source, asm in asm_of.items():
        for name, size in re.findall(r"\.amdhsa_kernel (\w+)\n(?:.*\n)*?\s*\.amdhsa_private_segment_fixed_size (\d+)", asm):
            kernels_seen += 1
            assert int(size) == 0, f"{source}: {name}: {size} bytes"
        assert not re.search(r"^\s*scratch_(load|store)", asm, re.M), source
    assert kernels_seen > 40
