"""What the sweep kernels rely on in the code that the compiler makes of them, read
from the disassembly of the built library (two conditions that no compiler check
covers, as the instructions concerned are inline assembly):
* the source of a DPP operand is not written by a vector instruction within the two
  wait states before it, on any path (an s_nop n counts n + 1);
* the 4 x 4 row pipeline publishes a tile's counter only when the wavefront's stores
  of it are drained: on every path from a store of the distribution to the counter's
  store lies a wait that as many later vector-memory operations make cover it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1712_01132_amd import build, poredvm

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")


class Insn:
    __slots__ = ("op", "args", "prev")

    def __init__(self, op, args):
        self.op, self.args, self.prev = op, args, []


def parse(lines):
    """The instructions of one kernel with their predecessors (falling through or
    branching). lines: (address, text, branch target or None)."""
    insns, at, jumps = [], {}, []
    for addr, text, target in lines:
        op, _, rest = text.partition(" ")
        i = Insn(op, [a.strip() for a in rest.split(",")] if rest else [])
        at[addr] = len(insns)
        if insns and insns[-1].op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            i.prev.append(len(insns) - 1)
        if target is not None:
            jumps.append((len(insns), target))
        insns.append(i)
    for src, target in jumps:
        insns[at[target]].prev.append(src)
    return insns


def regs(arg):
    m = re.match(r"v\[(\d+):(\d+)\]", arg)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)\b", arg)
    return {int(m[1])} if m else set()


def written(i):
    if not i.op.startswith("v_") or not i.args:
        return set()
    return regs(i.args[0]) | (regs(i.args[1]) if i.op.startswith("v_swap") else set())


def dpp_violations(insns):
    """Indices of DPP instructions whose source a vector instruction writes too late."""
    bad = []
    for n, i in enumerate(insns):
        if "_dpp" not in i.op:
            continue
        src = regs(i.args[1])
        todo = [(p, 0) for p in i.prev]
        seen = set()
        while todo:
            p, states = todo.pop()
            if states >= 2 or (p, states) in seen:
                continue
            seen.add((p, states))
            q = insns[p]
            if written(q) & src:
                bad.append(n)
                break
            states += int(q.args[0], 0) + 1 if q.op == "s_nop" else 1
            todo += [(r, states) for r in q.prev]
    return bad


def is_vmem(i):
    return re.match(r"(buffer|global|flat|scratch)_(load|store|atomic)", i.op) is not None


def counter_stores(insns):
    """The stores of the progress counters: the dword stores with sc1 to an address that
    the kernel never polls (the fault flag is polled)."""
    addr = lambda i: (i.args[2].split()[0], re.findall(r"offset:\S+", i.args[-1]))
    polled = [addr(i) for i in insns if i.op == "global_load_dword" and i.args[-1].endswith("sc1")]
    return [n for n, i in enumerate(insns)
            if i.op == "global_store_dword" and i.args[-1].endswith("sc1") and addr(i) not in polled]


def undrained(insns):
    """The counter stores that a store of the distribution can reach undrained. Per
    instruction: the fewest vector-memory operations issued since an undrained
    buffer_store, on any path (DRAINED if there is none)."""
    DRAINED = 1 << 20
    nxt = [[] for _ in insns]
    for n, i in enumerate(insns):
        for p in i.prev:
            nxt[p].append(n)
    before = [DRAINED] * len(insns)
    todo = [n for n, i in enumerate(insns) if i.op.startswith("buffer_store")]
    after = {}
    work = list(todo)
    while work:
        n = work.pop()
        i = insns[n]
        out = before[n]
        if i.op.startswith("buffer_store"):
            out = 0
        elif is_vmem(i) and out < 64:
            out += 1
        elif i.op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", ",".join(i.args))
            if m and out >= int(m[1]):
                out = DRAINED
        if after.get(n) == out:
            continue
        after[n] = out
        for k in nxt[n]:
            if out < before[k]:
                before[k] = out
                work.append(k)
    return [n for n in counter_stores(insns) if before[n] != DRAINED]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(poredvm.LIB_PATH):
        build.build()
    d = tmp_path_factory.mktemp("code")
    lib = os.path.join(d, "lib.so")
    shutil.copy(poredvm.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    out, lines = {}, None
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(d, f)], check=True, capture_output=True,
                              text=True).stdout
        for line in text.splitlines():
            m = re.match(r"([0-9a-f]+) <(.*)>:", line)
            if m:
                start = int(m[1], 16)
                lines = out.setdefault(m[2], []) if "sweep" in m[2] else None  # the others hold no such assembly
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and lines is not None:
                target = None
                if m[1].startswith(("s_branch", "s_cbranch")):
                    t = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>", m[3])
                    target = start + int(t[1] or "0", 16)
                lines.append((int(m[2], 16), m[1], target))
    return {k: parse(v) for k, v in out.items()}


def test_no_dpp_operand_is_written_too_late(kernels):
    n = 0
    for name, insns in kernels.items():
        bad = dpp_violations(insns)
        assert not bad, (name, [(insns[k].op, insns[k].args) for k in bad[:3]])
        n += sum("row_newbcast" in i.args[-1] for i in insns if i.args)
    assert n > 1000


def test_rows4_counters_follow_drained_stores(kernels):
    n = 0
    for name, insns in kernels.items():
        if "sweep_rows4_kernel" not in name:
            continue
        assert counter_stores(insns)
        assert not undrained(insns), name
        n += 1
    assert n == 24  # two precisions, two protocols, six model combinations


def test_the_checks_find_planted_faults():
    def code(*text):
        return parse([(4 * k, t, None) for k, t in enumerate(text)])

    dpp = "v_mov_b32_dpp v1, v2 row_newbcast:3 row_mask:0xf bank_mask:0xf"
    assert dpp_violations(code("v_mov_b32_e32 v2, v3", "s_nop 0", dpp)) == [2]
    assert dpp_violations(code("v_mov_b64_e32 v[2:3], v[4:5]", "s_nop 1", dpp)) == []
    loop = parse([(0, "s_nop 1", None), (4, dpp, None), (8, "v_mov_b32_e32 v2, v3", None), (12, "s_cbranch_scc1 4", 4)])
    assert dpp_violations(loop) == [1]

    store = "buffer_store_dword v1, v2, s[0:3], 0 offen"
    load = "global_load_dword v3, v4, s[4:5]"
    post = "global_store_dword v5, v6, s[8:9] sc1"
    assert undrained(code(store, load, load, load, "s_waitcnt vmcnt(4)", post)) == [5]
    assert undrained(code(store, load, load, load, load, "s_waitcnt vmcnt(4)", post)) == []
    assert undrained(code(load, load, load, load, store, "s_waitcnt vmcnt(4)", post)) == [6]
