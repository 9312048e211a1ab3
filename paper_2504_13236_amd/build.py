"""Builds libnntile_mi.so (the C-ABI library of HIP kernels for gfx950) in-tree.

    python -m paper_2504_13236_amd.build

Every .hip file under csrc/ is compiled with hipcc for gfx950 and linked into
paper_2504_13236_amd/libnntile_mi.so.  Works without a GPU (cross-compilation).
"""
from __future__ import annotations

import concurrent.futures
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libnntile_mi.so")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-fvisibility=hidden",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
    # packed fp32 VALU forms are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # per-kernel register, scratch and LDS figures on stderr (parsed below)
    "-Rpass-analysis=kernel-resource-usage",
]

# Sources whose kernels keep LDS reads in flight across statements (the reads are issued by
# inline assembly and waited for later by hand): a register the compiler spills or reloads
# between a read and its wait would hold stale data, so inside their loops these kernels
# must not touch scratch memory.  (Spills in the prologue or after the last wait are harmless.)
# Their assembly is also scanned for any instruction that names a register between the LDS read that
# targets it and the wait for it (registers_touched_in_flight): a copy or move the compiler
# places there would read stale data just the same.  Both follow the branches, not the order of the listing: loop blocks
# carry their loop's name on the line of their label or on the next one, and the compiler puts blocks out of line.
IN_FLIGHT_SOURCES = ("gemm_bf16_dl.hip", "gemm_bf16_span.hip", "gemm_f32_dl.hip")
# Sources with matrix instructions: their assembly is scanned for uses of a result before it is there.
MATRIX_SOURCES = IN_FLIGHT_SOURCES + ("gemm_bf16.hip", "gemm_f32.hip", "attention.hip")


_VREG = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")


def _vregs(text: str) -> set:
    out = set()
    for m in _VREG.finditer(text):
        if m.group(1) is not None:
            out.add(int(m.group(1)))
        else:
            out.update(range(int(m.group(2)), int(m.group(3)) + 1))
    return out


# Wait states (instructions, an `s_nop n` counting as n + 1) that have to lie between a matrix instruction and another
# kind of instruction that names its result: the hardware does not hold such an instruction back.  The numbers
# are those that the compiler leaves in straight-line code.
MATRIX_WAIT_STATES = {"v_mfma_f32_32x32x2_f32": 18, "v_mfma_f32_32x32x16_bf16": 12}
_ANYREG = re.compile(r"\b([va])(\d+)\b|\b([va])\[(\d+):(\d+)\]")


def _registers(text: str) -> set:
    out = set()
    for m in _ANYREG.finditer(text):
        if m.group(1):
            out.add((m.group(1), int(m.group(2))))
        else:
            out.update((m.group(3), r) for r in range(int(m.group(4)), int(m.group(5)) + 1))
    return out


def _kernels(asm_text: str) -> dict:
    """{kernel: ([(line number, instruction, operands)], {label: index of the instruction behind it})}."""
    out: dict = {}
    code = labels = None
    for no, line in enumerate(asm_text.splitlines(), 1):
        t = line.split(";")[0].strip()
        if t.endswith(":"):
            if t.startswith("_Z"):
                code, labels = out.setdefault(t[:-1], ([], {}))
            elif t.startswith(".Lfunc_end"):
                code = labels = None
            elif labels is not None:
                labels[t[:-1]] = len(code)
        elif t and code is not None and not t.startswith("."):
            op, _, rest = t.partition(" ") if " " in t else t.partition("\t")
            code.append((no, op, rest.strip()))
    return out


def _next(code: list, labels: dict, i: int) -> list:
    """Indices of the instructions that may follow instruction i."""
    _, op, args = code[i]
    if op == "s_endpgm" or op.startswith("s_setpc"):
        return []
    to = [labels[args]] if op == "s_branch" else [i + 1] + ([labels[args]] if op.startswith("s_cbranch") else [])
    return [j for j in to if j < len(code)]


def scratch_in_loops(asm_text: str) -> list:
    """[(kernel, line number)] of scratch instructions of a device assembly listing that can be reached from themselves."""
    hits = []
    for kernel, (code, labels) in _kernels(asm_text).items():
        for first, (no, op, _) in enumerate(code):
            if not op.startswith("scratch_"):
                continue
            seen, todo = set(), _next(code, labels, first)
            while todo:
                i = todo.pop()
                if i not in seen:
                    seen.add(i)
                    todo += _next(code, labels, i)
            if first in seen:
                hits.append((kernel, no))
    return hits


def registers_touched_in_flight(asm_text: str) -> list:
    """[(kernel, line number, register, line of the read)]: instructions of a device assembly listing that name a
    vector register while an LDS read into it is still in flight on a path that leads to them, i.e. between the ds_read that
    targets it and the `s_waitcnt lgkmcnt(n)` that covers it (LDS operations complete in order, so such a wait leaves at most
    the last n of them in flight; scalar loads only make a wait cover more than is assumed here).

    The compiler believes such a register holds its value from the read's asm statement on, so a copy, a move to
    an accumulation register or any other use it schedules before the hand-placed wait would see stale data."""
    hits = set()
    for kernel, (code, labels) in _kernels(asm_text).items():
        # in front of each instruction: register -> (LDS operations from its read on, the read included; line of the read),
        # the fewest where paths meet
        before: list = [None] * len(code)
        todo = []

        def reach(i, state):
            if before[i] is None:
                before[i] = dict(state)
                todo.append(i)
            else:
                newer = {r: p for r, p in state.items() if p < before[i].get(r, (1 << 30,))}
                if newer:
                    before[i].update(newer)
                    todo.append(i)

        if code:
            reach(0, {})
        while todo:
            i = todo.pop()
            no, op, args = code[i]
            state = dict(before[i])
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                if m:
                    state = {r: p for r, p in state.items() if p[0] <= int(m.group(1))}
            else:
                target = set()
                if op.startswith("ds_read"):            # its operands behind the first are the address, read now
                    ops = args.split(",")
                    target, args = _vregs(ops[0]), ",".join(ops[1:])
                hits.update((kernel, no, "v%d" % r, state[r][1]) for r in _vregs(args) if r in state)
                if op.startswith("ds_"):
                    state = {r: (n + 1, at) for r, (n, at) in state.items()}
                state.update((r, (1, no)) for r in target)
            for j in _next(code, labels, i):
                reach(j, state)
    return sorted(hits, key=lambda h: (h[0], h[1], int(h[2][1:])))


def matrix_results_named_early(asm_text: str) -> list:
    """[(kernel, line number, line of the matrix instruction, wait states between them)]: instructions of a device assembly
    listing that name the result of a matrix instruction before it is there, on any path through the branches.

    The compiler puts the wait states in itself, but counts them along one of the paths that meet in a block, which need
    not be the shortest.  Another matrix instruction with the same result is no such use: it is held back by the hardware,
    and what comes after it is looked at from there."""
    hits = set()
    for kernel, (code, labels) in _kernels(asm_text).items():
        for first, (no, op, rest) in enumerate(code):
            if not op.startswith(("v_mfma", "v_smfma")):
                continue
            if op not in MATRIX_WAIT_STATES:
                raise RuntimeError("%s: the wait states behind %s are not on record" % (kernel, op))
            result, best = _registers(rest.split(",")[0]), {}
            todo = [(first + 1, 0)]
            while todo:
                i, waited = todo.pop()
                while i < len(code) and waited < min(MATRIX_WAIT_STATES[op], best.get(i, 1 << 30)):
                    best[i] = waited
                    at, name, args = code[i]
                    if name.startswith("v_mfma"):
                        parts = args.split(",")
                        if _registers(parts[1] + "," + parts[2]) & result:
                            hits.add((kernel, at, no, waited))
                        if _registers(parts[0]) & result:
                            break
                    elif _registers(args) & result:
                        hits.add((kernel, at, no, waited))
                        break
                    waited += int(args, 0) + 1 if name == "s_nop" else 1
                    to = _next(code, labels, i)
                    if not to:
                        break
                    i = to[0]
                    todo += [(j, waited) for j in to[1:]]
    return sorted(hits)


_NAME = re.compile(r"remark: Function Name: (\S+)")
_FIELD = re.compile(r"remark:\s+(TotalSGPRs|VGPRs|AGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]"
                    r"|VGPRs Spill|LDS Size \[bytes/block\]): (\d+)")


def resource_usage(stderr: str) -> dict:
    """{mangled kernel name: {field: value}} from hipcc's kernel-resource-usage remarks."""
    out: dict = {}
    cur = None
    for line in stderr.splitlines():
        m = _NAME.search(line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = _FIELD.search(line)
        if m and cur is not None:
            cur[m.group(1).split(" [")[0]] = int(m.group(2))
    return out


def _newest_header() -> float:
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    hs += [os.path.join(ROOT, "include", f) for f in os.listdir(os.path.join(ROOT, "include"))]
    return max(os.path.getmtime(h) for h in hs)


def _compile(src: str, only_if_stale: bool = False) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    if only_if_stale and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), _newest_header(),
                                                                              os.path.getmtime(__file__)):
        return obj
    name = os.path.basename(src)
    cmd = ["hipcc", *FLAGS, *(["-save-temps=obj"] if name in MATRIX_SOURCES else []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr[-4000:]))
    usage = resource_usage(r.stderr)
    if name in MATRIX_SOURCES:
        with open(os.path.join(OBJ, os.path.splitext(name)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")) as f:
            asm = f.read()
        named = matrix_results_named_early(asm)
        if named:
            raise RuntimeError("%s: %s, assembly line %d, names the result of the matrix instruction of line %d after %d wait states (%d such uses in all)"
                               % (name, *named[0], len(named)))
    if name in IN_FLIGHT_SOURCES:
        hits = scratch_in_loops(asm)
        if hits:
            raise RuntimeError("%s: scratch access inside a loop of %s (assembly line %d, %d in all): "
                               "in-flight fragment registers do not survive a spill"
                               % (name, hits[0][0], hits[0][1], len(hits)))
        early = registers_touched_in_flight(asm)
        if early:
            raise RuntimeError("%s: %s, assembly line %d, uses %s before the wait for the LDS read of line %d (%d such uses in all)"
                               % (name, early[0][0], early[0][1], early[0][2], early[0][3], len(early)))
    with open(obj + ".usage.json", "w") as f:
        json.dump(usage, f, indent=1, sort_keys=True)
    return obj


def build_library(jobs: int | None = None, verbose: bool = True, only_stale: bool = False) -> str:
    """Compiles every source (or, with only_stale, those older than their object file) and links."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))
    jobs = jobs or min(8, len(srcs), os.cpu_count() or 1)
    with concurrent.futures.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda f: _compile(f, only_stale), srcs))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr[-4000:])
    if verbose:
        print("built", LIB, "from", len(srcs), "sources")
    return LIB


if __name__ == "__main__":
    build_library(only_stale="--stale" in sys.argv[1:])
    sys.exit(0)
