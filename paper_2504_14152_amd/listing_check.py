"""Static check of the compiled main loop of the prefill GEMM (no GPU needed).

The loop's global loads are inline assembly whose completion the compiler does
not track: a register that a load in flight will write must not be read or
written until a wait has guaranteed the load has landed.  Loads complete in
issue order, so `s_waitcnt vmcnt(N)` guarantees every load that has at least N
younger memory operations behind it.  The functions below read the gfx950
listing the build's own flags produce and verify that property instruction by
instruction, along every path through the kernel (a wait in one branch says
nothing about the others), and that the loop holds neither register spills nor a full
`vmcnt(0)` wait (the stall the assembly loads exist to avoid).  build() runs
check() on every build, with the compiler and flags of that build, and fails
the build if it trips; the tests call the same functions.
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

KERNELS = {
    "fp32 output": "_ZN4fgmp17gemm_mixed_kernelILi2ELi4ELb0ELb0EE",
    "packed output": "_ZN4fgmp17gemm_mixed_kernelILi2ELi4ELb1ELb0EE",
    "gated packed output": "_ZN4fgmp17gemm_mixed_kernelILi2ELi4ELb1ELb1EE",
}


def make_listing(hipcc: str, flags: list[str], src: str) -> list[str]:
    """The device-side assembly listing of `src` under the given build flags, as lines."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "listing.s")
        flags = [f for f in flags if f != "-fPIC"]
        res = subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", "-o", out, src], capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"listing of {src} failed:\n{res.stderr}")
        with open(out) as fh:
            return fh.read().split("\n")


def instructions(lines):
    return [l.strip() for l in lines if l.startswith("\t") and not l.strip().startswith((";", "."))]


def kernel_body(lines, prefix):
    start = next(i for i, l in enumerate(lines) if l.startswith(prefix) and ":" in l)
    end = next(i for i in range(start, len(lines)) if "s_endpgm" in lines[i])
    return lines[start:end]


def main_loop(body):
    hdr = next(i for i, l in enumerate(body) if "Inner Loop Header" in l)
    label = body[hdr].split(":")[0]
    back = next(i for i in range(hdr, len(body)) if re.search(r"s_(?:cbranch_\w+|branch)\s+" + re.escape(label) + r"\b", body[i]))
    return body[hdr + 1 : back + 1]


def _regs(text):
    out = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]", text):
        out.update(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r"\bv(\d+)\b", text):
        out.add(int(m.group(1)))
    return out


def _is_vmem(ins):
    return ins.startswith(("buffer_load", "buffer_store", "global_load", "global_store", "scratch_"))


def violations(ins, cyclic):
    """(number of loads checked, loads whose destination is touched before a wait has made them land)."""
    n = len(ins)
    bad = []
    checked = 0
    for i, s in enumerate(ins):
        if not s.startswith("buffer_load"):
            continue
        dst = _regs(s.split(",")[0])
        younger = 0
        landed = False
        span = range(1, 2 * n) if cyclic else range(1, n - i)
        for step in span:
            t = ins[(i + step) % n] if cyclic else ins[i + step]
            m = re.match(r"s_waitcnt.*vmcnt\((\d+)\)", t)
            if m and int(m.group(1)) <= younger:
                landed = True
            if _regs(t) & dst:
                checked += 1
                if not landed:
                    bad.append((s, t))
                break
            if _is_vmem(t):
                younger += 1
    return checked, bad


def whole_kernel(lines, prefix):
    """The lines of a kernel, blocks listed behind its first s_endpgm included."""
    start = next(i for i, l in enumerate(lines) if l.startswith(prefix) and ":" in l)
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return lines[start + 1 : end]


def flow_violations(body):
    """(number of loads to registers, touches of a destination that some path reaches with the load in flight).  Walks the
    control-flow graph of a kernel's lines: what is in flight at a label is what any way to it leaves in flight, with the fewest
    younger memory operations of all ways."""
    code, at = [], {}
    for l in body:
        label = re.match(r"(\.?\w+):", l)
        if label:
            at[label.group(1)] = len(code)
        elif instructions([l]):
            code.append(l.split(";")[0].strip())
    known = {}   # state in front of an instruction: register -> (younger memory operations, the load)
    bad = {}
    todo = [(0, {})]
    while todo:
        i, state = todo.pop()
        while i < len(code):
            seen = known.get(i)
            if seen is None:
                merged = dict(state)
            else:
                merged = dict(seen)
                for r, v in state.items():
                    if r not in merged or v[0] < merged[r][0]:
                        merged[r] = v
                if merged == seen:
                    break
            known[i] = merged
            state = dict(merged)
            ins = code[i]
            wait = re.match(r"s_waitcnt.*vmcnt\((\d+)\)", ins)
            if wait:
                state = {r: v for r, v in state.items() if v[0] < int(wait.group(1))}
            for r in _regs(ins) & state.keys():
                bad[(state[r][1], ins)] = None
                del state[r]   # (once is enough)
            if _is_vmem(ins):
                state = {r: (min(y + 1, 64), load) for r, (y, load) in state.items()}
                if re.match(r"(?:buffer|global|scratch)_load", ins) and not re.search(r"\blds\b|_lds_", ins):
                    state.update((r, (0, ins)) for r in _regs(ins.split(",")[0]))
            jump = re.match(r"s_(cbranch_\w+|branch)\s+(\.?\w+)", ins)
            if jump and jump.group(2) in at:
                todo.append((at[jump.group(2)], state))
            if ins.startswith("s_endpgm") or (jump and jump.group(1) == "branch"):
                break
            i += 1
    loads = sum(ins.startswith("buffer_load") and not re.search(r"\blds\b", ins) for ins in code)
    return loads, list(bad)


def direct_loads_without_wait(lines) -> tuple[int, list]:
    """(number of direct loads to LDS, those right behind the scalar instruction that writes M0).  M0 holds a direct load's
    LDS address; the instruction set asks for one instruction or s_nop between the two, and the compiler does not look
    inside inline assembly."""
    ins = instructions(lines)
    direct = [i for i, s in enumerate(ins) if re.match(r"(?:global|buffer|scratch)_load", s) and re.search(r"\blds\b|_lds_", s)]
    return len(direct), [(ins[i - 1], ins[i]) for i in direct if re.match(r"s_\w+ m0,", ins[i - 1])]


def check_kernel(lines, prefix) -> list[str]:
    """Problems found in one kernel of the listing (empty: none)."""
    problems = []
    body = kernel_body(lines, prefix)
    loop = instructions(main_loop(body))
    if sum(s.startswith("v_mfma") for s in loop) != 6 * 32:
        problems.append("the loop body is not one turn of the register rotation (6 K-steps of 32 matrix instructions)")
    checked, bad = violations(loop, cyclic=True)
    if checked < 6 * 6 or bad:
        problems.append(f"main loop: {checked} loads checked, hazards {bad}")
    checked, bad = flow_violations(whole_kernel(lines, prefix))   # prologue -> loop -> remainder -> epilogue
    if checked < 60 or bad:
        problems.append(f"whole kernel: {checked} loads checked, hazards {bad}")
    if [s for s in loop if s.startswith("scratch_")]:
        problems.append("register spill inside the main loop")
    waits = [int(m.group(1)) for s in loop for m in [re.match(r"s_waitcnt.*vmcnt\((\d+)\)", s)] if m]
    if not waits or min(waits) < 6:
        problems.append(f"a wait in the main loop drains (nearly) all loads: {waits}")
    return problems


MID_KERNEL = "_ZN4fgmp15gemm_mid_kernel"


def mid_kernels(lines) -> list[str]:
    """The instantiations of the kernel for a few dozen to a few hundred rows in a listing."""
    return [l.split(":")[0] for l in lines if l.startswith(MID_KERNEL) and ":" in l]


def k_loop(body):
    """The loop that holds matrix instructions (its header may be listed behind its first pass)."""
    for hdr in (i for i, l in enumerate(body) if "Loop Header" in l):
        label = body[hdr].split(":")[0]
        back = [i for i in range(hdr, len(body)) if re.search(r"s_(?:cbranch_\w+|branch)\s+" + re.escape(label) + r"\b", body[i])]
        if back and any("v_mfma" in l for l in body[hdr : back[-1] + 1]):
            return body[hdr + 1 : back[-1] + 1]
    raise RuntimeError("no loop with matrix instructions")


def check_mid_kernel(lines, name) -> list[str]:
    """The same for one instantiation gemm_mid_kernel<MT, NT, WN, WK>: two rounds per turn of its loop, two waits per round."""
    mt, nt, wn, _ = (int(v) for v in re.search(r"ILi(\d)ELi(\d)ELi(\d)ELi(\d)E", name).groups())
    problems = []
    body = kernel_body(lines, name)
    loop = instructions(k_loop(body))
    if sum(s.startswith("v_mfma") for s in loop) != 2 * 4 * mt * nt:
        problems.append("the loop body is not two rounds of four quarters")
    checked, bad = violations(loop, cyclic=True)
    if checked != 2 * 5 * nt or bad:
        problems.append(f"main loop: {checked} loads checked, hazards {bad}")
    checked, bad = flow_violations(whole_kernel(lines, name))
    if checked < 4 * 5 * nt or bad:
        problems.append(f"whole kernel: {checked} loads checked, hazards {bad}")
    if [s for s in loop if s.startswith("scratch_")]:
        problems.append("register spill inside the main loop")
    waits = [int(m.group(1)) for s in loop for m in [re.match(r"s_waitcnt.*vmcnt\((\d+)\)", s)] if m]
    if waits != 2 * [4 * mt // wn, 5 * nt]:
        problems.append(f"waits in the main loop: {waits}")
    return problems


def check_mid(hipcc: str, flags: list[str], src: str) -> None:
    """Raise if any instantiation of gemm_mid_kernel, compiled as the build compiles it, has a hazard."""
    lines = make_listing(hipcc, flags, src)
    found = {n: p for n in mid_kernels(lines) for p in [check_mid_kernel(lines, n)] if p}
    if direct_loads_without_wait(lines)[1]:
        found["direct loads"] = direct_loads_without_wait(lines)[1]
    if found or not mid_kernels(lines):
        raise RuntimeError(f"gemm_mid_kernel listing check failed: {found}")


def check(hipcc: str, flags: list[str], src: str) -> None:
    """Raise if any instantiation of the prefill kernel, compiled as the build compiles it, has a hazard."""
    lines = make_listing(hipcc, flags, src)
    found = {}
    for name, prefix in KERNELS.items():
        p = check_kernel(lines, prefix)
        if p:
            found[name] = p
    if direct_loads_without_wait(lines)[1]:
        found["direct loads"] = direct_loads_without_wait(lines)[1]
    if found:
        raise RuntimeError(f"prefill kernel listing check failed: {found}")
