"""Builds libmoe355.so (all HIP sources, gfx950) next to this file with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmoe355.so")
SOURCES = ["api.hip", "route.hip", "permute.hip", "ffn.hip", "ffn_f32.hip", "combine.hip", "schedule.hip"]
# ffn.hip is compiled in parts, side by side: each of its large kernels is an object of its own.
PARTS = {"ffn.hip": 5}
UNITS = [(src, part) for src in SOURCES for part in range(PARTS.get(src, 1))]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


# ffn.hip spells out its software pipeline (loads first, LDS reads one k-step ahead of the MFMAs); the
# machine scheduler would fold that back into load-use pairs to save registers, so it is switched off there.
# Its work-queue atomics are issued by one lane whose answer is wanted later (it arrives under other work); the atomic
# optimizer would rewrite them into a wave reduction whose broadcast waits for the answer on the spot.
EXTRA = {"ffn.hip": ["-mllvm", "-enable-misched=false", "-mllvm", "-amdgpu-atomic-optimizer-strategy=None"]}
# The MFMA kernels of ffn.hip keep loads in flight in registers the compiler knows nothing about and count
# the outstanding loads by hand.  Spill code inside such a region could save a register before its load
# has landed, and its own memory operations would be counted as if they were the kernel's.  The source
# brackets those regions with "; pipeline begin" / "; pipeline end"; the build reads the assembly and
# refuses any scratch access between the two or inside an inner loop of these kernels.
NO_SPILL = {"ffn.hip": "ffn_mfma"}
# The parts of ffn.hip with tiles of more than 16 blocks, whose last sums are in assembly.
TALL = (1, 3, 4)


def check_no_spill(asm: str, kernel_pattern: str, what: str = "assembly") -> None:
    """Raises if a kernel whose name contains kernel_pattern touches scratch memory between a
    "; pipeline begin" and the next "; pipeline end", or inside a loop nested in another loop."""
    kernel, inside, inner = None, False, False
    lines = asm.splitlines()
    for n, line in enumerate(lines, 1):
        text = line.strip()
        if line.startswith("_Z") and ":" in line:                       # a function starts
            name = line.split(":")[0]
            kernel = name if kernel_pattern in name else None
            inside = inner = False
        elif text.startswith(".end_amdhsa_kernel") or text.startswith(".Lfunc_end"):
            kernel = None
        if kernel is None:
            continue
        if line.startswith(".LBB") or line.startswith("; %bb."):        # a block: which loop is it in?
            note = line + (lines[n] if n < len(lines) and lines[n].strip().startswith(";") else "")
            inner = "Depth=2" in note or "Depth=3" in note
        if "; pipeline begin" in text:
            inside = True
        elif "; pipeline end" in text:
            inside = False
        elif text.startswith("scratch_") and (inside or inner):
            raise RuntimeError(f"{what}: spill code inside a hand-counted load pipeline of {kernel} (line {n}: {text})")



_VREG = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def _vregs(text: str) -> set:
    out = set()
    for lo, hi, one in _VREG.findall(text):
        out |= set(range(int(lo), int(hi) + 1)) if lo else {int(one)}
    return out


def _load_dst(text: str) -> set:
    """Registers a vector memory load writes: its first operand, or none (a load into LDS, whose first operand is an address)."""
    return set() if "_lds_" in text.split()[0] else _vregs(text.split(",")[0])


def check_loads_in_flight(asm: str, kernel_pattern: str, what: str = "assembly") -> int:
    """The pipelined loops of the named kernels keep loads in flight that the compiler does not know about
    (it sees inline assembly that defines registers).  Whatever it schedules or copies there, no instruction
    may touch a register whose load has not been waited for.  This walks every inner loop that lies between
    "; pipeline begin" and "; pipeline end", twice around (the second round meets the loads the first left in
    flight), keeping the loads in issue order: "s_waitcnt vmcnt(N)" retires all but the youngest N (loads
    return in order), and any other use of a register with a load still pending is an error.  The loops must
    be single blocks.  Returns the number of loops checked."""
    lines = asm.splitlines()
    kernel, inside, checked, n = None, False, 0, 0
    while n < len(lines):
        line = lines[n]
        text = line.strip()
        if line.startswith("_Z") and ":" in line:
            name = line.split(":")[0]
            kernel = name if kernel_pattern in name else None
            inside = False
        elif text.startswith(".end_amdhsa_kernel"):
            kernel = None
        if kernel is not None:
            if "; pipeline begin" in text:
                inside = True
            elif "; pipeline end" in text:
                inside = False
            elif inside and line.startswith(".LBB") and "Depth=2" in (line + (lines[n + 1] if n + 1 < len(lines) else "")):
                label = line.split(":")[0]
                body, m = [], n + 1
                while m < len(lines):
                    t = lines[m].strip()
                    if lines[m].startswith(".LBB") or "; pipeline" in t:
                        raise RuntimeError(f"{what}: the pipelined loop {label} of {kernel} is not a single block (line {m + 1})")
                    if t and not t.startswith(";"):
                        body.append((m + 1, t.split(";")[0].strip()))
                    if t.startswith("s_cbranch") and t.split()[-1] == label:
                        break
                    m += 1
                pending = []                                  # (registers, line) in issue order
                for round_ in range(2):
                    for ln, t in body:
                        op = t.split()[0]
                        if op == "s_waitcnt":
                            got = re.search(r"vmcnt\((\d+)\)", t)
                            if got:
                                keep = int(got.group(1))
                                pending = pending[len(pending) - keep:] if 0 < keep < len(pending) else ([] if keep == 0 else pending)
                            continue
                        used = _vregs(t)
                        for regs, at in pending:
                            if used & regs:
                                raise RuntimeError(f"{what}: {kernel}: line {ln} ({t}) touches v{min(used & regs)}, whose load "
                                                   f"(line {at}) has not been waited for")
                        if op.startswith(("global_load", "buffer_load", "flat_load")):
                            pending.append((_load_dst(t), ln))
                checked += 1
                n = m
        n += 1
    return checked


def check_m0_free(asm: str, kernel_pattern: str, what: str = "assembly") -> int:
    """The loads into LDS set m0 in the inline assembly that issues them.  The register is a reserved one, which a clobber list cannot
    name; so no instruction of the named kernels outside of inline assembly may touch it, else it would find the loads' value there or they
    its.  Raises on one; returns the number of lines of inline assembly that write it."""
    kernel, in_asm, written = None, False, 0
    for n, line in enumerate(asm.splitlines(), 1):
        text = line.strip()
        if line.startswith("_Z") and ":" in line:
            name = line.split(":")[0]
            kernel = name if kernel_pattern in name else None
        elif text.startswith((".end_amdhsa_kernel", ".Lfunc_end")):
            kernel = None
        if text.startswith((";;#ASMSTART", ";;#ASMEND")):
            in_asm = text.startswith(";;#ASMSTART")
        elif kernel is not None and re.search(r"\bm0\b", text.split(";")[0]):
            if not in_asm:
                raise RuntimeError(f"{what}: {kernel}: line {n} ({text}) touches m0, which the loads into LDS set without the compiler's knowledge")
            written += 1
    return written


_SUM = re.compile(r"v_mfma\S+ v\[(\d+):(\d+)\], ([^,]+), ([^,]+), (\S+)")
_SETTLE = 18                             # wait states after which the longest of these instructions has written its sum


def check_sums_settle(asm: str, kernel_pattern: str, what: str = "assembly") -> int:
    """The sums that do not fit the accumulation registers come from matrix instructions in inline assembly, whose latency the compiler
    does not know.  Nothing but the same kind of instruction, as its sum, may touch such registers before _SETTLE wait states have passed
    (an instruction is one, "s_nop N" N + 1), on any way the program can take from there; and no vector instruction may have written one of its operands
    in the two wait states before it, in layout order.  Raises on either; returns the number of those instructions."""
    lines = asm.splitlines()
    labels = {l.split(":")[0]: i for i, l in enumerate(lines) if l.startswith(".LBB")}
    kernel, in_asm, found, now, written = None, False, 0, 0, {}      # written: register -> wait state after the last vector instruction that wrote it

    def walk(at, sum_of, passed):                      # from line `at` on, `passed` wait states after the instruction
        regs = set(range(sum_of[0], sum_of[1] + 1))
        while at < len(lines) and passed < _SETTLE:
            text = lines[at].strip().split(";")[0].strip()
            at += 1
            if text.startswith(".Lfunc_end"):
                return
            if not text or text.startswith(".") or text.endswith(":"):
                continue
            got = _SUM.match(text)
            whole = got is not None and (int(got[1]), int(got[2])) == sum_of and got[5] == f"v[{got[1]}:{got[2]}]"
            if (_vregs(got[3] + "," + got[4]) if whole else _vregs(text)) & regs:
                raise RuntimeError(f"{what}: {kernel}: line {at} ({text}) touches v[{sum_of[0]}:{sum_of[1]}] {passed} wait states after a matrix instruction in assembly")
            if whole or text.startswith("s_endpgm"):
                return                                 # (the next one of this sum is looked at by itself)
            op = text.split()[0]
            passed += int(text.split()[1], 0) + 1 if op == "s_nop" else 1
            if op.startswith(("s_branch", "s_cbranch")):
                if text.split()[-1] not in labels:
                    raise RuntimeError(f"{what}: {kernel}: line {at} ({text}) goes to an unknown place")
                walk(labels[text.split()[-1]], sum_of, passed)
                if op == "s_branch":
                    return
            elif op.startswith(("s_setpc", "s_swappc", "s_call")):
                raise RuntimeError(f"{what}: {kernel}: line {at} ({text}) goes to an unknown place")

    for n, line in enumerate(lines):
        text = line.strip()
        if line.startswith("_Z") and ":" in line:
            name = line.split(":")[0]
            kernel, written = (name if kernel_pattern in name else None), {}
        elif text.startswith((".end_amdhsa_kernel", ".Lfunc_end")):
            kernel = None
        if text.startswith((";;#ASMSTART", ";;#ASMEND")):
            in_asm = text.startswith(";;#ASMSTART")
        code = text.split(";")[0].strip()
        if kernel is None or not code or code.startswith(".") or code.endswith(":"):
            continue
        got = _SUM.match(code)
        if in_asm and got:
            early = [reg for reg in _vregs(code) if now - written.get(reg, -2) < 2]
            if early:
                raise RuntimeError(f"{what}: {kernel}: line {n + 1} ({code}) reads v{early[0]} within two wait states of its writing")
            found += 1
            walk(n + 1, (int(got[1]), int(got[2])), 0)
        now += int(code.split()[1], 0) + 1 if code.startswith("s_nop") else 1
        if code.startswith("v_") and not got:
            written.update((reg, now) for reg in _vregs(code.split(",")[0]))
    return found


def check_prologue_in_flight(asm: str, kernel_pattern: str, what: str = "assembly") -> int:
    """The same rule for the code that leads up to each pipelined loop (from "; pipeline begin" to the loop's
    first block, in layout order, across block labels): the loads written as inline assembly are in flight from
    their issue until a "s_waitcnt vmcnt(N)" that leaves at most N younger ones outstanding, and nothing may
    touch their registers before.  Vector memory operations the compiler generated itself in that stretch
    (one wave takes the block's next work item there) are not put on the list: a wave that does not execute
    them has fewer operations outstanding, so counting them would retire hand-issued loads too early.
    Returns the number of stretches checked."""
    lines = asm.splitlines()
    kernel, checked, n = None, 0, 0
    while n < len(lines):
        line = lines[n]
        if line.startswith("_Z") and ":" in line:
            name = line.split(":")[0]
            kernel = name if kernel_pattern in name else None
        elif line.strip().startswith(".end_amdhsa_kernel"):
            kernel = None
        if kernel is not None and "; pipeline begin" in line:
            pending, in_asm, m = [], True, n + 1          # the marker itself is inline assembly
            while m < len(lines):
                raw = lines[m]
                t = raw.strip()
                if "; pipeline end" in t:
                    break
                if raw.startswith(".LBB") and "Depth=2" in (raw + (lines[m + 1] if m + 1 < len(lines) else "")):
                    break
                if "#ASMSTART" in t:
                    in_asm = True
                elif "#ASMEND" in t:
                    in_asm = False
                if t and not t.startswith(";") and not raw.startswith("."):
                    code = t.split(";")[0].strip()
                    op = code.split()[0]
                    if op == "s_waitcnt":
                        got = re.search(r"vmcnt\((\d+)\)", code)
                        if got:
                            keep = int(got.group(1))
                            pending = pending[len(pending) - keep:] if 0 < keep < len(pending) else ([] if keep == 0 else pending)
                    else:
                        used = _vregs(code)
                        for regs, at in pending:
                            if used & regs:
                                raise RuntimeError(f"{what}: {kernel}: line {m + 1} ({code}) touches v{min(used & regs)}, whose "
                                                   f"load (line {at}) has not been waited for")
                        if in_asm and op.startswith(("global_load", "buffer_load", "flat_load")):
                            pending.append((_load_dst(code), m + 1))
                m += 1
            checked += 1
            n = m
        n += 1
    return checked


def _flags(src: str, part: int) -> list:
    return [*FLAGS, *EXTRA.get(src, []), *([f"-DFFN_PART={part}"] if src in PARTS else [])]


def _built(src: str, part: int, suffix: str) -> str:
    return os.path.join(HERE, "_build", src.replace(".hip", f"_{part}{suffix}" if src in PARTS else suffix))


def _check(src: str, part: int) -> None:
    """Compiles the unit to assembly and refuses what the checks above refuse (ffn.hip's part 0 holds no pipelined loop)."""
    asm = _built(src, part, ".s")
    ra = subprocess.run([_hipcc(), *_flags(src, part), "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", asm],
                        capture_output=True, text=True)
    if ra.returncode != 0:
        raise RuntimeError(f"hipcc -S failed on {src}:\n{ra.stderr}")
    text = open(asm).read()
    check_no_spill(text, NO_SPILL[src], src)
    loops = check_loads_in_flight(text, NO_SPILL[src], src), check_prologue_in_flight(text, NO_SPILL[src], src)
    m0 = check_m0_free(text, NO_SPILL[src], src)
    sums = check_sums_settle(text, NO_SPILL[src], src)
    if part > 0 and (0 in loops or m0 == 0):
        raise RuntimeError(f"{src}: no pipelined loop, or no load into LDS, found to verify (markers missing?)")
    if part in TALL and sums == 0:
        raise RuntimeError(f"{src}, part {part}: no matrix instruction in assembly found to verify (printed in another way?)")


def _compile(src: str, part: int) -> str:
    obj = _built(src, part, ".o")
    cmd = [_hipcc(), *_flags(src, part), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as pool:
        checks = [pool.submit(_check, src, part) for src, part in UNITS if src in NO_SPILL]
        objs = list(pool.map(lambda u: _compile(*u), UNITS))
        for c in checks:
            c.result()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
