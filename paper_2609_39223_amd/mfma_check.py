"""Wait states around the MFMAs that the NT GEMM writes as inline assembly (csrc/qf_gemm_nt.hip).

The compiler keeps the wait states that gfx950 wants from software only around MFMAs it knows; the
NT GEMM's are inline assembly, whose correctness rests on where the register allocator puts copies.
check_library() disassembles those kernels in a built library and fails if, along any path,
  - a vector instruction writes a register that an MFMA reads less than 2 wait states later, or
  - anything but an MFMA that accumulates onto the same registers accesses an MFMA's result less
    than 18 wait states later (16x16x32 bf16: eight passes).
An instruction is one wait state, s_nop n is n + 1.
"""
import glob
import os
import re
import shutil
import subprocess
import tempfile

KERNELS = ("gemm_nt_kernel", "gemm_nt_rows_kernel")
VALU_TO_MFMA = 2
MFMA_TO_ANY = 18

_REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
_LINE = re.compile(r"^\s+(\S+)(.*?)\s*//\s*([0-9A-Fa-f]+):")
_HEAD = re.compile(r"^([0-9a-f]+) <(\S+)>:")
_TARGET = re.compile(r"<\S+\+0x([0-9a-f]+)>\s*$")


def _regs(text):
    out = []
    for m in _REG.finditer(text):
        lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
        out.extend((m[1], i) for i in range(lo, hi + 1))
    return out


def _operands(text):
    return [o.strip() for o in re.split(r",(?![^\[]*\])", text)]


class _Instruction:
    __slots__ = ("name", "text", "address", "target", "wait", "mfma", "writes", "reads")

    def __init__(self, name, text, address, target):
        self.name, self.text, self.address, self.target = name, text, address, target
        self.wait = int(text.strip() or "0", 0) + 1 if name == "s_nop" else 1
        self.mfma = name.startswith(("v_mfma", "v_smfmac"))
        ops = _operands(text)
        both = name.startswith(("v_swap", "v_permlane16_swap", "v_permlane32_swap"))
        if name.startswith("v_"):
            self.writes = _regs(ops[0]) + (_regs(ops[1]) if both else [])
            self.reads = [_regs(o) for o in (ops if both else ops[1:])]
        else:                                   # memory and LDS: a load's registers count as access
            self.writes = []
            self.reads = [_regs(o) for o in ops]


def parse(listing):
    """{function: [instructions]} of an llvm-objdump listing."""
    functions, cur, start = {}, None, 0
    for line in listing.splitlines():
        h = _HEAD.match(line)
        if h:
            start, cur = int(h[1], 16), functions.setdefault(h[2], [])
            continue
        m = _LINE.match(line)
        if cur is None or not m:
            continue
        target = None
        if m[1].startswith(("s_branch", "s_cbranch")):
            t = _TARGET.search(line)
            target = start + int(t[1], 16) if t else start
        cur.append(_Instruction(m[1], m[2], int(m[3], 16), target))
    return functions


def _blocks(code):
    index = {c.address: i for i, c in enumerate(code)}
    leaders = {0}
    for i, c in enumerate(code):
        if c.target is not None or c.name == "s_endpgm":
            leaders.add(i + 1)
        if c.target is not None:
            leaders.add(index[c.target])
    leaders = sorted(x for x in leaders if x < len(code))
    blocks = []
    for n, a in enumerate(leaders):
        b = leaders[n + 1] if n + 1 < len(leaders) else len(code)
        last, succ = code[b - 1], []
        if last.target is not None:
            succ.append(index[last.target])
        if last.name not in ("s_branch", "s_endpgm") and b < len(code):
            succ.append(b)
        blocks.append((a, b, succ))
    return blocks


def hazards(code):
    """Messages for the instructions of one function that come too soon after a write."""
    blocks = _blocks(code)
    at = {a: n for n, (a, _, _) in enumerate(blocks)}
    entry = [None] * len(blocks)                # {(register, by MFMA): wait states since}
    entry[0] = {}
    found, work = {}, [0]
    while work:
        a, b, succ = blocks[work.pop()]
        since = {k: -v for k, v in entry[at[a]].items()}   # the time of the write, plus one
        now = 0
        for i in range(a, b):
            c = code[i]
            for n, group in enumerate(c.reads):
                for r in group:
                    if c.mfma and now - since.get((r, False), -MFMA_TO_ANY) < VALU_TO_MFMA:
                        found[i] = "reads %s%d too soon after a vector write" % r
                    onto = c.mfma and n == 2 and group == c.writes
                    if not onto and now - since.get((r, True), -MFMA_TO_ANY) < MFMA_TO_ANY:
                        found[i] = "reads %s%d too soon after an MFMA" % r
            for r in c.writes:
                if not c.mfma and now - since.get((r, True), -MFMA_TO_ANY) < MFMA_TO_ANY:
                    found[i] = "writes %s%d too soon after an MFMA" % r
                if c.name.startswith("v_"):
                    since.pop((r, not c.mfma), None)
                    since[(r, c.mfma)] = now + 1
            now += c.wait
        out = {k: now - v for k, v in since.items() if now - v < MFMA_TO_ANY}
        for s in succ:
            n = at[s]
            old = entry[n]
            new = dict(out) if old is None else dict(old)
            for k, v in out.items():
                new[k] = min(v, new.get(k, v))
            if old is None or new != old:
                entry[n] = new
                work.append(n)
    return ["%x: %s%s: %s" % (code[i].address, code[i].name, code[i].text, found[i])
            for i in sorted(found)]


def kernels(path, objdump):
    """[(name, instructions)] of the kernels with inline-assembly MFMAs in a built library."""
    found = []
    with tempfile.TemporaryDirectory() as tmp:
        lib = shutil.copy(path, os.path.join(tmp, "lib.so"))
        subprocess.run([objdump, "--offloading", lib], cwd=tmp, check=True, capture_output=True)
        for obj in glob.glob(os.path.join(tmp, "lib.so.*gfx950*")):
            r = subprocess.run([objdump, "-d", "--no-show-raw-insn", obj], check=True,
                               capture_output=True, text=True)
            found += [(name, code) for name, code in parse(r.stdout).items()
                      if any(k in name for k in KERNELS) and any(c.mfma for c in code)]
    return found


def check_library(path, objdump):
    """Number of kernels checked; raises RuntimeError on a hazard or if there is none to check."""
    checked = kernels(path, objdump)
    bad = ["%s: %s" % (name, h) for name, code in checked for h in hazards(code)]
    if not checked:
        raise RuntimeError("no GEMM kernel found in %s" % path)
    if bad:
        raise RuntimeError("MFMA hazards in %s:\n%s" % (path, "\n".join(bad[:20])))
    return len(checked)
