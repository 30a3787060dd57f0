"""Static check of the built library's machine code (developer tool; nothing at run time uses it).

The compiler inserts the wait states that the hardware leaves to software between the instructions it emits itself, but it does
not look into inline assembly, and much of this package's device code issues its loads there.  This script disassembles
the gfx950 code of libelitekv.so (which this repository built) and follows every kernel's control flow, so it holds for
whatever the compiler made of the sources, whoever wrote the instruction:

  sgpr   a vector-memory instruction that reads a scalar register (an address, a buffer descriptor, an offset) fewer than five wait
         states after a vector instruction wrote it (v_readfirstlane and the like) may use the register's old value
  m0     a direct-to-LDS load right behind the write of M0, which holds its place in the LDS, may go to the place before it; one
         wait state must lie between
  query  a register of the split attention's query is read, or given to something else, before the load that fills it has landed

    python -m paper_2503_01586_amd.check_machine_code [libelitekv.so]

Every finding is printed with its kernel and address; exit status 1 if there are any.
"""
from __future__ import annotations

import collections
import os
import re
import shutil
import subprocess
import sys
import tempfile

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(PKG_DIR, "libelitekv.so")
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")

SGPR_WAIT = 5
M0_WAIT = 1
MOST_BEHIND = 63                                           # a wave has no more than 63 vector-memory operations under way
MEMORY = ("global_", "buffer_", "flat_", "scratch_")
# registers as integers: v0.. from 0, a0.. from 1000, s0.. from 2000, then the named ones
BASE = {"v": 0, "a": 1000, "s": 2000}
NAMED = {"vcc": (3000, 3001), "vcc_lo": (3000,), "vcc_hi": (3001,), "m0": (3002,)}
M0 = NAMED["m0"][0]
_REG = re.compile(r"\b(?:([vas])(?:(\d+)|\[(\d+):(\d+)\])|(vcc_lo|vcc_hi|vcc|m0))(?![\w\[])")
_CODE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+): ([0-9A-F ]+)")
_VMCNT = re.compile(r"vmcnt\((\d+)\)")
_LABEL = re.compile(r"^[0-9a-f]+ <([^>]+)>:")

Finding = collections.namedtuple("Finding", "rule kernel address text what")


def scalar(reg: int) -> bool:
    return reg >= 2000


def registers(text: str) -> tuple:
    out = []
    for kind, one, lo, hi, named in _REG.findall(text):
        if named:
            out += NAMED[named]
        elif one:
            out.append(BASE[kind] + int(one))
        else:
            out += range(BASE[kind] + int(lo), BASE[kind] + int(hi) + 1)
    return tuple(out)


class Instruction:
    __slots__ = ("address", "op", "text", "operands", "states", "target")

    def __init__(self, op, text, address, code):
        self.op, self.address, self.text = op, address, op + " " + text
        self.operands = [registers(t) for t in text.split(",")]
        self.states = int(text, 0) + 1 if op == "s_nop" else 1           # wait states it stands for
        self.target = None
        if op.startswith(("s_branch", "s_cbranch")):
            low = int(code.split()[0], 16) & 0xffff
            self.target = address + 4 + 4 * (low - 0x10000 if low & 0x8000 else low)

    @property
    def memory(self) -> bool:
        return self.op.startswith(MEMORY)

    def written_scalars(self) -> tuple:
        """Scalar registers that a vector instruction writes: the first operand's, or a carry's or scale's in the second."""
        if not self.op.startswith("v_"):
            return ()
        two = "_co_" in self.op or self.op.startswith(("v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32"))
        return tuple(r for t in self.operands[:2 if two else 1] for r in t if scalar(r))


def disassemble(lib: str):
    """(kernel name, its instructions) of every gfx950 code object in the library."""
    with tempfile.TemporaryDirectory(prefix="ekv_isa_") as tmp:
        copy = shutil.copy(lib, tmp)                       # the code objects are written beside the file
        subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True, cwd=tmp)
        for f in sorted(os.listdir(tmp)):
            if not f.endswith("gfx950"):
                continue
            text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp, f)], check=True, capture_output=True, text=True).stdout
            name, code = None, []
            for line in text.splitlines():
                label = _LABEL.match(line)
                if label:
                    if code:
                        yield name, code
                    name, code = label.group(1), []
                    continue
                m = _CODE.match(line)
                if m:
                    code.append(Instruction(m.group(1), m.group(2), int(m.group(3), 16), m.group(4)))
            if code:
                yield name, code


def blocks_of(code):
    """Basic blocks of a kernel: lists of instructions, and the numbers of the blocks that may follow each."""
    leaders = {code[0].address}
    for i, ins in enumerate(code):
        if ins.target is not None or ins.op == "s_endpgm":
            if ins.target is not None:
                leaders.add(ins.target)
            if i + 1 < len(code):
                leaders.add(code[i + 1].address)
    blocks, number = [], {}
    for ins in code:
        if ins.address in leaders:
            number[ins.address] = len(blocks)
            blocks.append([])
        blocks[-1].append(ins)
    follow = []
    for i, b in enumerate(blocks):
        last, nxt = b[-1], []
        if last.target is not None:
            nxt.append(number[last.target])
        if last.op not in ("s_branch", "s_endpgm") and i + 1 < len(blocks):
            nxt.append(i + 1)
        follow.append(nxt)
    return blocks, follow


class Scan:
    """State: register -> wait states since the write that is looked for; the fewest over all ways that lead here."""

    def __init__(self, rule, wait, what):
        self.rule, self.wait, self.what = rule, wait, what

    def merge(self, old, state):
        """Takes `state` into the entry state `old` of a block; whether that changed it."""
        changed = False
        for r, n in state.items():
            if old.get(r, self.wait) > n:
                old[r], changed = n, True
        return changed

    def run(self, kernel, blocks, follow):
        entry = [None] * len(blocks)
        entry[0] = {}
        work = [0]
        while work:
            i = work.pop()
            state = dict(entry[i])
            for ins in blocks[i]:
                self.step(state, ins)
            for j in follow[i]:
                if entry[j] is None:
                    entry[j] = dict(state)
                    work.append(j)
                elif self.merge(entry[j], state) and j not in work:
                    work.append(j)
        findings = []
        for i, b in enumerate(blocks):
            if entry[i] is None:
                continue
            state = dict(entry[i])
            for ins in b:
                early = [n for r in self.reads(ins) for n in (state.get(r),) if n is not None]
                if early:
                    findings.append(Finding(self.rule, kernel, ins.address, ins.text, self.what % min(early)))
                self.step(state, ins)
        return findings

    def step(self, state, ins):
        for r in [r for r, n in state.items() if n + ins.states >= self.wait]:
            del state[r]
        for r in state:
            state[r] += ins.states
        for r in self.writes(ins):
            state[r] = 0
        for r in self.settled(ins):
            state.pop(r, None)


class VectorWrittenScalars(Scan):
    def __init__(self):
        super().__init__("sgpr", SGPR_WAIT, "reads a scalar register %%d wait states after a vector instruction wrote it (%d needed)"
                         % SGPR_WAIT)

    def reads(self, ins):
        return tuple(r for t in ins.operands for r in t if scalar(r)) if ins.memory else ()

    def writes(self, ins):
        return ins.written_scalars()

    def settled(self, ins):                                # written anew by the scalar unit: no vector write is waited for
        return ins.operands[0] if ins.op.startswith("s_") and not ins.op.startswith(("s_cmp", "s_bitcmp", "s_cbranch")) else ()


class LdsLoadsBehindM0(Scan):
    def __init__(self):
        super().__init__("m0", M0_WAIT, "reads M0 %%d wait states after it was written (%d needed)" % M0_WAIT)

    def reads(self, ins):
        return (M0,) if ins.memory and ("_load_lds_" in ins.op or ins.text.endswith(" lds")) else ()

    def writes(self, ins):
        return (M0,) if M0 in ins.operands[0] and not ins.op.startswith(("s_cmp", "s_bitcmp")) else ()

    def settled(self, ins):
        return ()


class QueryInFlight:
    """The split attention issues its query loads ahead of the first tile's wait; until then nothing may touch their registers:
    a read finds the old value, and what is written there (the registers are free wherever the query is not used, in
    an empty split) is overwritten when the load lands.  Followed from the blocks that load the query to the first matrix
    product or to the wait that covers a load: vmcnt(n) does where n other operations were issued behind it, for they complete in
    order (the most of all the ways that lead there: which tiles were requested is not followed).  A way that leads from one
    such block to another is left out: a launch loads the query once."""
    rule, what = "query", "uses a register that a load of the query has yet to fill"

    def run(self, kernel, blocks, follow):
        if "attn_mfma_kernel" not in kernel:
            return []
        product = next(ins for b in blocks for ins in b if ins.op.startswith("v_mfma"))
        loads = [[k for k, ins in enumerate(b) if self.loads(ins) and set(product.operands[2]) & set(ins.operands[0])]
                 for b in blocks]
        before = collections.defaultdict(list)
        for i, nxt in enumerate(follow):
            for j in nxt:
                before[j].append(i)
        once, work = set(), [i for i, b in enumerate(blocks) if b[-1].op == "s_endpgm"]
        while work:                                        # blocks from which the end is reached without loading (again)
            i = work.pop()
            if i not in once and not loads[i]:
                once.add(i)
                work += before[i]
        findings = {}
        for i, at in enumerate(loads):
            if at:
                self.follow(kernel, blocks, follow, once, i, findings)
        assert any(loads), kernel
        return [findings[a] for a in sorted(findings)]

    @staticmethod
    def loads(ins):
        return ins.op == "global_load_dwordx4" and ins.text.endswith(", off")

    def follow(self, kernel, blocks, follow, once, start, findings):
        entry, work = {start: {}}, [start]                 # register -> operations issued behind its load
        while work:
            i = work.pop()
            live = dict(entry[i])
            for ins in blocks[i]:
                if ins.op.startswith("v_mfma"):
                    live.clear()
                    break
                if ins.op == "s_waitcnt":
                    n = _VMCNT.search(ins.text)
                    live = {r: behind for r, behind in live.items() if n is None or behind < int(n.group(1))}
                    continue
                load = i == start and self.loads(ins)
                if any(r in live for t in ins.operands[1 if load else 0:] for r in t):
                    findings[ins.address] = Finding(self.rule, kernel, ins.address, ins.text, self.what)
                if ins.memory:
                    live = {r: min(behind + 1, MOST_BEHIND) for r, behind in live.items()}
                if load:
                    live.update((r, 0) for r in ins.operands[0])
            for j in follow[i]:
                if live and j in once:
                    old = entry.setdefault(j, {})
                    more = {r: behind for r, behind in live.items() if behind > old.get(r, -1)}
                    if more:
                        old.update(more)
                        work.append(j)


SCANS = (VectorWrittenScalars(), LdsLoadsBehindM0(), QueryInFlight())


def check(lib: str = LIB_PATH, scans=SCANS):
    """(kernels scanned, findings)."""
    kernels, findings = 0, []
    for name, code in disassemble(lib):
        kernels += 1
        blocks, follow = blocks_of(code)
        for scan in scans:
            findings += scan.run(name, blocks, follow)
    return kernels, findings


def main(argv):
    kernels, findings = check(*argv[1:2])
    for f in findings:
        print("%s: %s %x: %s: %s" % (f.rule, f.kernel, f.address, f.text, f.what))
    print("%d kernels scanned, %d findings in %d of them" % (kernels, len(findings), len({f.kernel for f in findings})))
    return 1 if findings else 0


if __name__ == "__main__":
    sys.exit(main(sys.argv))
