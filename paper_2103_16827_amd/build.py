"""Builds libqasr.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqasr.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
    # packed-fp32 instruction forms are kept off on this platform
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results stay in ordinary vector registers (no copies through the accumulator file)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-command-line-argument",
    # per-kernel register / scratch / LDS figures as compiler remarks: kept in resource_usage.txt
    "-Rpass-analysis=kernel-resource-usage",
]
RESOURCES = os.path.join(HERE, "resource_usage.txt")


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip"))) + sorted(glob.glob(os.path.join(CSRC, "*.cpp")))


def kernels_using_scratch(recs):
    """Names of the kernels whose resource record (name, then `Key:value` strings as the compiler
    printed them, blanks removed) does not say `ScratchSize[bytes/lane]:0`."""
    return [r[0] for r in recs if "ScratchSize[bytes/lane]:0" not in r[1:]]


def partial_write_hazards(asm_text: str):
    """Instruction pairs in device assembly where a vector instruction reads a register that the
    instruction just before it wrote through a byte/word selector (`..._sdwa` with `dst_sel` other
    than DWORD).  gfx950 needs one instruction in between; the compiler inserts it for its own
    code but cannot see inside `asm` statements."""
    ins = []
    for l in asm_text.splitlines():
        l = l.strip()
        if not l or l[0] in ";./" or l.endswith(":"):
            continue
        ins.append(l)
    bad = []
    for a, b in zip(ins, ins[1:]):
        if "_sdwa" in a.split()[0] and "dst_sel:" in a and "dst_sel:DWORD" not in a:
            dst = a.split()[1].rstrip(",")
            if b.startswith("v_") and re.search(r"\b" + re.escape(dst) + r"\b", b):
                bad.append((a, b))
    return bad


def _registers(operands: str):
    """Numbers of the vector registers named in an operand list."""
    regs = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", operands):
        regs |= {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))
    return regs


def _kernels(asm_text: str):
    """(name, instructions, successors) of every function in device assembly: each instruction with whether an `asm` statement
    put it there, and the indexes of those that can run right after it."""
    for part in re.split(r"\n(?=_Z\w+:)", asm_text)[1:]:
        ins, at, by_hand = [], {}, False
        for line in part.split(".Lfunc_end")[0].splitlines()[1:]:
            line = line.strip()
            label = re.match(r"(\.L\w+):", line)
            if label:
                at[label.group(1)] = len(ins)
            elif "#ASMSTART" in line or "#ASMEND" in line:
                by_hand = "#ASMSTART" in line
            elif line and line[0] not in ";." and not line.endswith(":"):
                ins.append((line.split(";")[0].strip(), by_hand))
        after = []
        for i, (text, _) in enumerate(ins):
            jump = re.match(r"s_(c?branch)\w*\s+(\.L\w+)", text)
            nxt = [] if text.startswith("s_endpgm") or (jump and jump.group(1) == "branch") else [i + 1]
            after.append([j for j in nxt + ([at[jump.group(2)]] if jump else []) if j < len(ins)])
        yield part.split(":")[0], ins, after


def _reached(starts, after):
    """Indexes that can run after one of `starts` has."""
    seen, todo = set(), [j for i in starts for j in after[i]]
    while todo:
        i = todo.pop()
        if i not in seen:
            seen.add(i)
            todo += after[i]
    return seen


def _copies_out_of(text: str):
    """Registers that an instruction copies from (none if it is no copy)."""
    return _registers(text.partition(",")[2]) if re.match(r"v_(mov|accvgpr|swap|pk_mov)", text) else set()


def ring_copies(asm_text: str):
    """(kernel, instruction) for every copy, after one matrix product and before another on some path, out of a register that a
    hand-issued 16-byte load fills which can have run before, further up or an iteration earlier.  To the compiler such a
    register holds its value from the `asm` statement on, so it may move it while the load is on its way (it has, where it indexed a ring at run time): the copy is then
    what was there before, and the data lands in a register that belongs to something else."""
    bad = []
    for name, ins, after in _kernels(asm_text):
        products = [i for i, (text, _) in enumerate(ins) if text.startswith("v_mfma")]
        before = [[] for _ in ins]
        for i, nxt in enumerate(after):
            for j in nxt:
                before[j].append(i)
        between = _reached(products, after) & _reached(products, before)
        ring = {}                                     # register -> its loads
        for i, (text, by_hand) in enumerate(ins):
            if by_hand and re.match(r"(global|buffer)_load_dwordx4 ", text):
                for r in _registers(text.split(",")[0]):
                    ring.setdefault(r, []).append(i)
        later = {}                                    # ... -> what can run after one of them
        for i in sorted(between):
            for r in _copies_out_of(ins[i][0]) & set(ring):
                if r not in later:
                    later[r] = _reached(ring[r], after)
                if i in later[r]:
                    bad.append((name, ins[i][0]))
                    break
    return bad


def copies_in_flight(asm_text: str):
    """(kernel, instruction) for every copy out of a register whose hand-issued load (of any size) need not have completed on
    some path, wherever in the kernel it stands.  Loads complete in the order of their requests: one is complete after
    `vmcnt(N)` if at least N requests came after it."""
    bad = []
    for name, ins, after in _kernels(asm_text):
        state = [None] * len(ins)                     # at each instruction: register -> fewest requests after its load
        todo = [0] if ins else []
        if ins:
            state[0] = {}
        while todo:
            i = todo.pop()
            text, by_hand = ins[i]
            out = dict(state[i])
            wait = re.match(r"s_waitcnt\b.*vmcnt\((\d+)\)", text)
            if wait:
                out = {r: n for r, n in out.items() if n < int(wait.group(1))}
            if re.match(r"v_|(ds|global|buffer|flat|scratch)_(read|load)", text) and not by_hand:
                for r in _registers(text.split(",")[0]):   # (another value from here on)
                    out.pop(r, None)
            if re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", text):
                out = {r: min(n + 1, 63) for r, n in out.items()}
                if by_hand and "_load_" in text and "_lds_" not in text:
                    out.update(dict.fromkeys(_registers(text.split(",")[0]), 0))
            for j in after[i]:
                new = dict(state[j] or {})
                for r, n in out.items():
                    new[r] = min(n, new.get(r, 63))
                if new != state[j]:
                    state[j] = new
                    todo.append(j)
        bad += [(name, text) for i, (text, _) in enumerate(ins) if state[i] and _copies_out_of(text) & set(state[i])]
    return bad


def source_with_local_includes(src: str, seen=None) -> str:
    """Text of a source file followed by that of every header of this directory it includes."""
    seen = set() if seen is None else seen
    if src in seen or not os.path.exists(src):
        return ""
    seen.add(src)
    with open(src) as f:
        text = f.read()
    for inc in re.findall(r'#include\s+"([^"]+)"', text):
        text += source_with_local_includes(os.path.join(os.path.dirname(src), inc), seen)
    return text


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    procs = []
    asm_sources = []
    for src in sources():
        obj = os.path.join(bdir, os.path.basename(src) + ".o")
        cmd = [hipcc, "-x", "hip", "-c", src, "-o", obj] + [f for f in HIPCC_FLAGS if f != "-shared"]
        with open(src) as f:
            rings = re.search(r"gload16(_into\b|\()", f.read())
        if rings or "_sdwa" in source_with_local_includes(src):   # rings of hand-issued loads, hand-written partial register writes: device assembly too
            asm = os.path.join(bdir, os.path.basename(src) + ".gfx950.s")
            acmd = [hipcc, "-x", "hip", "--cuda-device-only", "-S", src, "-o", asm] + \
                   [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-Rpass-analysis=kernel-resource-usage")]
            asm_sources.append((src, asm, subprocess.Popen(acmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    remarks = []
    for src, pr in procs:
        out, _ = pr.communicate()
        remarks += [l for l in out.splitlines() if "[-Rpass-analysis=kernel-resource-usage]" in l]
        kept, skip = [], 0
        for l in out.splitlines():
            if "kernel-resource-usage" in l:
                skip = 2                       # the remark's echo of the source line and its caret
            elif skip and (l.lstrip().startswith("|") or "|" in l[:8]):
                skip -= 1
            elif "packed-fp32-ops" not in l and l.strip():
                kept.append(l)
        out = "\n".join(kept)
        if pr.returncode != 0:
            failed = True
            print(f"--- {src} failed:\n{out}", file=sys.stderr)
        elif out and verbose:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    # one line per kernel: name, then the figures the compiler reported for it
    recs, cur = [], None
    for l in remarks:
        body = l.split("remark:", 1)[1].replace("[-Rpass-analysis=kernel-resource-usage]", "").strip()
        if body.startswith("Function Name:"):
            cur = [body[len("Function Name:"):].strip()]
            recs.append(cur)
        elif cur is not None and ":" in body:
            cur.append(body.replace(" ", ""))
    with open(RESOURCES, "w") as f:
        for r in recs:
            f.write(" ".join(r) + "\n")
    # The pipelined kernels count their own vector-memory requests; a spill adds requests nobody
    # counted and moves registers that loads in flight still own.  Such a build must never run.
    for src, asm, pr in asm_sources:
        out, _ = pr.communicate()
        if pr.returncode != 0:
            raise RuntimeError(f"no device assembly for {src}:\n{out}")
        with open(asm) as f:
            text = f.read()
        for what, bad in (("register read right after a partial write", partial_write_hazards(text)),
                          ("copy of a register whose load may be on its way", ring_copies(text) or copies_in_flight(text))):
            if bad:
                if os.path.exists(LIB):
                    os.remove(LIB)
                raise RuntimeError(f"{asm}: {what}: {bad[0][0]} | {bad[0][1]}")
        os.remove(asm)
    if not recs:       # no figures parsed (the remark's format changed?): nothing was checked
        if os.path.exists(LIB):
            os.remove(LIB)
        raise RuntimeError("the compiler reported no per-kernel resource usage: the scratch-memory check cannot run")
    spilled = kernels_using_scratch(recs)
    if spilled:
        if os.path.exists(LIB):
            os.remove(LIB)
        raise RuntimeError("kernels use scratch memory (register spills): " + ", ".join(spilled))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
