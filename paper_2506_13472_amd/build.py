"""Builds librosaq.so (host packer + C ABI + gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import functools
import heapq
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "librosaq.so")
HOST_SOURCES = ["rosaq_pack.cpp", "rosaq_api.cpp"]
HIP_SOURCES = ["rosaq_kernels.hip", "rosaq_pca.hip", "rosaq_static.hip", "rosaq_quant.hip", "rosaq_rotate.hip",
               "rosaq_wide.hip"]


def hipcc() -> str:
    env = os.environ.get("HIPCC")
    if env:
        return env
    return "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


# The switch that keeps the compiler from forming packed-fp32 instructions is a feature of the gfx950
# target.  hipcc hands -Xclang options to its host pass as well, which does not know the feature and
# says so once per function-multiversioning probe; that line is dropped from the log.  What the
# device pass did is checked instead: its assembly (kept by -save-temps) must hold no packed-fp32
# arithmetic at all.
_HOST_NOISE = "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)"
_PK_F32 = re.compile(r"\bv_pk_(?:add|mul|fma)_f32\b")


# rosaq_wide.hip fetches LDS buffers ahead with hand-written loads and waits by count: in front of the pieces of a unit
# (four loads into LDS), "all but the N youngest loads are done", where the N youngest are two units' loads of weights and
# one unit's pieces.  How many loads of weights a unit has is the compiler's doing, so the assembly is counted.  A loop runs
# over two units, after and before a wait for everything: 0 L..L W DDDD L..L W DDDD L..L 0, with the loads behind
# the last pieces belonging to the first unit of the next turn.
_WAIT_LOOP = re.compile(r"0(L*)W(\d+)D{4}(L*)W(\d+)D{4}(L*)0")


def check_counted_waits(assembly: str) -> int:
    """The number of loops found; raises where one of their waits would not cover what it is there for, and where code
    of the compiler's uses m0, which the hand-written loads change without its knowledge."""
    events, in_asm = [], False
    for line in assembly.splitlines():
        op = line.strip()
        if op.startswith(";;#ASM"):
            in_asm = op.startswith(";;#ASMSTART")
        elif not in_asm and re.search(r"\bm0\b", op.split(";")[0]):
            raise RuntimeError(f"m0 outside the hand-written loads: {op}")
        elif "global_load_lds" in op:
            events.append("D")
        elif re.match(r"(global|flat|buffer)_load", op):
            events.append("L")
        elif in_asm and (m := re.match(r"s_waitcnt vmcnt\((\d+)\)$", op)):
            events.append("0" if m.group(1) == "0" else "W" + m.group(1))
    loops = _WAIT_LOOP.findall("".join(events))
    for head, first, middle, second, tail in loops:
        for loads, wait in ((len(head) + len(tail), int(first)), (len(middle), int(second))):
            if 2 * loads + 4 < wait:
                raise RuntimeError(f"vmcnt({wait}) counts on {(wait - 4) // 2} loads of weights in a unit, there are {loads}")
    return len(loops)


# A vector, LDS or memory instruction may touch the registers of an MFMA under way only after so many wait states (one per
# instruction, n + 1 for an s_nop n): a matrix instruction's result, whatever it is that touches it, and the sum that it
# starts from, if a vector instruction writes there.  The hardware does not wait by itself.  The compiler counts for
# the code that it makes, but it counts past a join of branches along one of the ways only, and inline assembly not at
# all.  So the assembly is searched along every way.  The figures are what the compiler keeps in straight code.
_MFMA_STATES = {            # (vector instruction at the result, LDS / memory instruction at it, vector write to the sum)
    "v_mfma_f32_16x16x32_f16": (8, 8, 3),
    "v_mfma_f64_16x16x4_f64": (19, 18, 0),
    "v_mfma_f32_16x16x4_f32": (10, 10, 7),
}
_REGISTERS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
_TOUCHES = ("v_", "ds_", "global_", "buffer_", "flat_", "scratch_")


def _registers(operands: str) -> frozenset:
    return frozenset((kind, i) for kind, lo, hi, one in _REGISTERS.findall(operands)
                     for i in range(int(one or lo), int(one or hi) + 1))


def check_mfma_distance(assembly: str) -> int:
    """The number of MFMAs found; raises where the way from one to an instruction that touches its registers is short."""
    program, labels = [], {}
    for line in assembly.splitlines():
        text = line.split(";")[0].split("//")[0].strip()
        if text.endswith(":"):
            labels[text[:-1]] = len(program)
        elif text and not text.startswith("."):
            op, _, operands = text.replace("\t", " ").partition(" ")
            program.append((op, operands.strip()))

    def successors(i):
        op, operands = program[i]
        if op == "s_branch":
            return (labels[operands],)
        if op == "s_endpgm":
            return ()
        if op in ("s_setpc_b64", "s_swappc_b64"):
            raise RuntimeError(f"{op}: a way that cannot be followed")
        after = (i + 1,) if i + 1 < len(program) else ()
        return after + (labels[operands],) if op.startswith("s_cbranch") else after

    @functools.lru_cache(maxsize=None)
    def uses(i):                                   # (all registers, registers that a vector instruction writes)
        op, operands = program[i]
        if not op.startswith(_TOUCHES):
            return frozenset(), frozenset()
        written = operands if "swap" in op else operands.split(", ")[0]
        return _registers(operands), _registers(written) if op.startswith("v_") else frozenset()

    found = 0
    for i, (op, operands) in enumerate(program):
        if not op.startswith("v_mfma"):
            continue
        if op not in _MFMA_STATES:
            raise RuntimeError(f"{op}: no wait states on file")
        found += 1
        vector, memory, write = _MFMA_STATES[op]
        parts = [_registers(t) for t in operands.split(", ")[:4]]
        result, summand = parts[0], parts[3]
        seen, ways = set(), [(0, j) for j in successors(i)]
        while ways:
            states, j = heapq.heappop(ways)
            if j in seen or states >= max(vector, memory, write):
                continue
            seen.add(j)
            other, other_operands = program[j]
            touched, written = uses(j)
            if other.startswith("v_mfma"):         # the sum of the next product may be this one's result; its factors may not
                touched, written = frozenset().union(*(_registers(t) for t in other_operands.split(", ")[1:3])), frozenset()
            need = vector if other.startswith("v_") else memory
            if (states < need and touched & result) or (states < write and written & summand):
                raise RuntimeError(f"{states} wait states between {op} {operands} and {other} {other_operands}")
            more = 1 + int(other_operands, 0) if other == "s_nop" else 1
            for k in successors(j):
                heapq.heappush(ways, (states + more, k))
    return found


def _compile_hip(src: str, obj: str, common, verbose: bool) -> None:
    cmd = [hipcc(), "-x", "hip", "--offload-arch=gfx950", "-save-temps=obj",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           *common, "-Wno-unused-command-line-argument", "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    log = [ln for ln in r.stdout.splitlines() if ln.strip() and ln.strip() != _HOST_NOISE]
    if log:
        print("\n".join(log), flush=True)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)
    stem = os.path.splitext(os.path.basename(obj))[0]            # e.g. rosaq_kernels.hip
    stem = os.path.splitext(stem)[0]
    asm = [f for f in os.listdir(os.path.dirname(obj))
           if f.startswith(stem + "-hip-amdgcn") and f.endswith(".s")]
    if not asm:
        raise RuntimeError(f"no device assembly kept for {src}")
    n = 0
    for f in asm:
        with open(os.path.join(os.path.dirname(obj), f), "r", errors="replace") as fh:
            text = fh.read()
        n += len(_PK_F32.findall(text))
        check_mfma_distance(text)
        if stem == "rosaq_wide" and check_counted_waits(text) != 3:      # INT4, INT3 and fp16
            raise RuntimeError(f"{src}: the counted waits of the LDS ring are not where they are looked for")
    print(f"{os.path.basename(src)}: device pass for gfx950 holds {n} packed-fp32 instructions", flush=True)
    if n:
        raise RuntimeError(f"{src}: packed-fp32 arithmetic in the device code")


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    common = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC,
              "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    jobs = []
    objs = []
    for s in HOST_SOURCES:
        o = os.path.join(OBJ, s + ".o")
        jobs.append((_run, ([hipcc(), "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-pthread", *common,
                             "-c", os.path.join(CSRC, s), "-o", o], verbose)))
        objs.append(o)
    for s in HIP_SOURCES:
        o = os.path.join(OBJ, s + ".o")
        jobs.append((_compile_hip, (os.path.join(CSRC, s), o, common, verbose)))
        objs.append(o)
    # the translation units are independent: compile them side by side
    with ThreadPoolExecutor(max_workers=min(len(jobs), max(1, (os.cpu_count() or 2) // 2))) as ex:
        for f in [ex.submit(fn, *a) for fn, a in jobs]:
            f.result()
    _run([hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-pthread", *objs, "-o", LIB], verbose)
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB)
