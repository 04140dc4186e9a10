"""Compile the HIP sources under csrc/ for gfx950 into libmoda.so next to this file."""
import glob
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmoda.so")
# the seeded input generator is a library of its own (it holds none of the operator's arithmetic)
SYNTH_SRC = os.path.join(HERE, "synth_csrc", "moda_synth.hip")
SYNTH_LIB = os.path.join(HERE, "libmoda_synth.so")

# the calls of binding.py in native code: a CPython module (host code only) against torch's headers
BIND_SRC = os.path.join(HERE, "bind_csrc", "moda_torch.cpp")
BIND_LIB = os.path.join(HERE, "moda_torch.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
    # compiler-generated packed fp32 math is switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True,
                   stderr=subprocess.PIPE if os.environ.get("MODA_QUIET_BUILD") else None)
    return obj


# Sources whose inline assembly owns ALL accumulation registers by name (see
# csrc/moda_fwd_regs.h) between the points where the kernel emits the marker comments
# ACC_ACQUIRE_MARKER and ACC_RELEASE_MARKER.  The compiler is not told that they hold live
# values, so the build verifies on the generated assembly, per kernel and on its
# control-flow graph, that
#   - no instruction that can execute between the two markers touches an accumulation
#     register unless it sits inside one of the hand-written assembly statements,
#   - no hand-written statement that names an accumulation register can execute before
#     the acquire marker or after the release marker (there the registers are the compiler's),
#   - nothing uses the result of a hand-written matrix instruction too early,
#   - nothing was spilled to scratch memory.
NAMED_ACC_SOURCES = ("moda_fwd_bf16.hip",)
ACC_ACQUIRE_MARKER = "MODA_ACC_REGISTERS_ACQUIRED"
ACC_RELEASE_MARKER = "MODA_ACC_REGISTERS_RELEASED"


def _kernel_bodies(asm_path):
    """Yields (name, [(line_no, text)]) for every function of the assembly file."""
    import re

    name, body = None, []
    for n, line in enumerate(open(asm_path), 1):
        if name is None:
            m = re.match(r"^(_Z\w+):", line)
            if m:
                name, body = m.group(1), []
        elif line.startswith(".Lfunc_end"):
            yield name, body
            name = None
        else:
            body.append((n, line.rstrip("\n")))


def _instructions(body):
    """The instruction stream of a function, [(line_no, text, hand_written)], with the markers as
    instructions of their own, and its labels, {name: index}."""
    import re

    ins, labels, in_asm = [], {}, False
    for n, line in body:
        if "#ASMSTART" in line:
            in_asm = True
            continue
        if "#ASMEND" in line:
            in_asm = False
            continue
        if in_asm and (ACC_RELEASE_MARKER in line or ACC_ACQUIRE_MARKER in line):
            ins.append((n, ACC_RELEASE_MARKER if ACC_RELEASE_MARKER in line else ACC_ACQUIRE_MARKER, True))
            continue
        code = line.split(";")[0].strip()
        if not code:
            continue
        m = re.match(r"^(\.LBB\d+_\d+):", code)
        if m:
            labels[m.group(1)] = len(ins)
            continue
        if code.startswith("."):
            continue
        ins.append((n, code, in_asm))
    return ins, labels


def _successors(asm_path, ins, labels, i):
    """Indices of the instructions that can execute right after instruction i."""
    op = ins[i][1].split()[0]
    if op in ("s_setpc_b64", "s_swappc_b64", "s_call_b64") or op.startswith("s_cbranch_i_fork"):
        raise RuntimeError("%s:%d: indirect control flow: %s" % (asm_path, ins[i][0], ins[i][1]))
    if op == "s_endpgm":
        return []
    if op == "s_branch":
        return [labels[ins[i][1].split()[1]]]
    out = [i + 1] if i + 1 < len(ins) else []
    if op.startswith("s_cbranch"):
        out.append(labels[ins[i][1].split()[1]])
    return out


# The compiler keeps other instructions away from a matrix instruction's result for as long as it takes, but not
# from the result of one that is written as inline assembly, and the hardware does not wait either: such a
# result (v_mfma_f32_32x32x16_bf16, 8 passes) may be read or overwritten no earlier than RESULT_SLOTS issue
# slots later, except by a matrix instruction that accumulates in the same registers.  A matrix instruction
# issued in between counts MFMA_SLOTS, s_nop N counts N + 1, any other one 1.
RESULT_SLOTS = 12
MFMA_SLOTS = 8


def _registers(text):
    """The vector and accumulation registers that an operand text names, as {("v" or "a", number)}."""
    import re

    out = set()
    for file, lo, hi, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update((file, r) for r in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    return out


def _check_result_distance(asm_path, name, body) -> None:
    ins, labels = _instructions(body)
    regs = [_registers(code) for _, code, _ in ins]

    def slots(i):
        op = ins[i][1].split()
        if op[0].startswith("v_mfma"):
            return MFMA_SLOTS
        return int(op[1], 0) + 1 if op[0] == "s_nop" else 1

    for start, (n, code, hand) in enumerate(ins):
        if not (hand and code.startswith("v_mfma")):
            continue
        result = _registers(code.split(None, 1)[1].split(",")[0])
        nearest, todo = {}, [(j, 0) for j in _successors(asm_path, ins, labels, start)]
        while todo:
            i, passed = todo.pop()
            if passed >= RESULT_SLOTS or nearest.get(i, RESULT_SLOTS) <= passed:
                continue
            nearest[i] = passed
            if regs[i] & result:
                operands = ins[i][1].split(None, 1)[1].split(", ") if ins[i][1].startswith("v_mfma") else []
                if len(operands) >= 4 and _registers(operands[0]) == result and not (
                        (_registers(operands[1]) | _registers(operands[2])) & result):
                    continue  # accumulates on; its own result is looked at in turn
                raise RuntimeError("%s:%d: %s: the result of line %d is used %d issue slots after it instead of %d: %s"
                                   % (asm_path, ins[i][0], name, n, passed, RESULT_SLOTS, ins[i][1]))
            todo.extend((j, passed + slots(i)) for j in _successors(asm_path, ins, labels, i))


def _check_kernel(asm_path, name, body) -> None:
    import re

    acc = re.compile(r"\ba(?:\[\d+:\d+\]|\d+)\b")
    ins, labels = _instructions(body)

    def the_marker(text):
        found = [i for i, x in enumerate(ins) if x[1] == text]
        if len(found) != 1:
            raise RuntimeError("%s: %s: expected exactly one %s, found %d" % (asm_path, name, text, len(found)))
        return found[0]

    acquire, marker = the_marker(ACC_ACQUIRE_MARKER), the_marker(ACC_RELEASE_MARKER)

    def successors(i):
        return _successors(asm_path, ins, labels, i)

    def reach(start, stop=None):
        seen, todo = set(), [start]
        while todo:
            i = todo.pop()
            if i in seen or i == stop:
                continue
            seen.add(i)
            todo.extend(successors(i))
        return seen

    if marker in reach(0, stop=acquire):
        raise RuntimeError("%s: %s: the release marker can be reached without passing the acquire marker"
                           % (asm_path, name))
    owned = reach(acquire, stop=marker)     # can execute between the markers
    free = reach(0, stop=acquire) | reach(marker)  # before the acquire marker or after the release marker
    for i in sorted(owned):
        n, code, hand = ins[i]
        if not hand and acc.search(code):
            raise RuntimeError("%s:%d: %s: compiler-allocated accumulation register while the named "
                               "ones are live: %s" % (asm_path, n, name, code))
    for i in sorted(free):
        n, code, hand = ins[i]
        if hand and acc.search(code):
            raise RuntimeError("%s:%d: %s: named accumulation register used outside the owned region: %s"
                               % (asm_path, n, name, code))


def check_named_acc_registers(src) -> None:
    asm = os.path.join(OBJ, os.path.basename(src)[:-4] + ".s")
    subprocess.run([HIPCC, *FLAGS, "--cuda-device-only", "-S", src, "-o", asm], check=True,
                   stderr=subprocess.DEVNULL)
    n_kernels = 0
    for name, body in _kernel_bodies(asm):
        _check_kernel(asm, name, body)
        _check_result_distance(asm, name, body)
        n_kernels += 1
    if n_kernels == 0:
        raise RuntimeError("%s: no kernel found" % asm)
    for line in open(asm):
        if line.startswith("; ScratchSize:") and int(line.split(":")[1]) != 0:
            raise RuntimeError("%s: register spill to scratch memory (%s)" % (asm, line.strip()))


# A loop that keeps global -> LDS copies or slot loads in flight while it computes must not touch
# scratch memory: memory operations complete in order, so waiting for a reload also waits for the
# copies (measured on the dK/dV kernel: 1.9 ms with 100 bytes of scratch per lane reloaded in the
# loop, 1.55 ms without).  Every kernel of every source is held to it, in each loop that encloses
# matrix instructions at any depth (the loop over positions around them is such a loop too) and, where
# a kernel has no matrix instructions, in each loop.  A value parked in scratch before the loops and
# fetched after them is harmless.


def check_no_scratch_in_loops(src) -> None:
    asm = os.path.join(OBJ, os.path.basename(src)[:-4] + ".s")
    subprocess.run([HIPCC, *FLAGS, "--cuda-device-only", "-S", src, "-o", asm], check=True,
                   stderr=subprocess.DEVNULL)
    scan_scratch_in_key_loops(asm)


def scan_scratch_in_key_loops(asm, name_part="") -> None:
    """Raises if a kernel of assembly file `asm` whose name contains `name_part` touches scratch
    memory inside a loop that encloses matrix instructions (any loop, if it has none)."""
    import re

    found = 0
    for name, body in _kernel_bodies(asm):
        if name_part not in name:
            continue
        found += 1
        # the compiler annotates every basic block of a loop with the header of its innermost loop,
        # and the header of a nested loop with the loops around it
        header, per_line, parent = None, [], {}
        block, around = None, {}
        for n, line in body:
            m = re.match(r"^(?:\.L(BB\d+_\d+):|; %bb\.\d+:)", line)
            if m:
                block, header, around = m.group(1), None, {}
            elif not re.match(r"^\s*;", line):
                block = None  # (the annotations of a block stand in the comment lines at its label)
            if m or block:
                around.update((int(d), h) for h, d in re.findall(r"Parent Loop (BB\d+_\d+) Depth=(\d+)", line))
                inside = re.search(r"in Loop: Header=(BB\d+_\d+)", line)
                if inside:
                    header = inside.group(1)
                elif "Loop Header" in line:
                    header = block
                    parent[block] = around[max(around)] if around else None
            per_line.append((n, line, header))
        has_mfma = any(re.match(r"^\s*v_mfma", line) for _, line, _ in per_line)
        hot = set()
        for _, line, h in per_line:
            if h and (not has_mfma or re.match(r"^\s*v_mfma", line)):
                while h and h not in hot:
                    hot.add(h)
                    h = parent.get(h)
        for n, line, h in per_line:
            # (a loop inside a hot one runs as often)
            while h and h not in hot:
                h = parent.get(h)
            if h and re.match(r"^\s*scratch_", line):
                raise RuntimeError("%s:%d: %s touches scratch memory inside a key loop: %s"
                                   % (asm, n, name, line.strip()))
    if found == 0 and name_part:
        raise RuntimeError("%s: no kernel named *%s*" % (asm, name_part))


def build_libmoda() -> str:
    """Always recompiles every source, then links.  Returns the library path."""
    os.makedirs(OBJ, exist_ok=True)
    for src in sources():
        if os.path.basename(src) in NAMED_ACC_SOURCES:
            check_named_acc_registers(src)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        checks = [ex.submit(check_no_scratch_in_loops, src) for src in sources()]
        objs = list(ex.map(_compile, sources()))
        for c in checks:
            c.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    build_synth()
    build_binding()
    return LIB


def build_binding() -> str:
    """Compiles the native half of the binding into moda_torch.so (g++; no device code)."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    rocm = os.path.dirname(os.path.dirname(HIPCC))
    inc = [x for d in (*include_paths(), sysconfig.get_paths()["include"], os.path.join(rocm, "include"))
           for x in ("-isystem", d)]
    libs = [x for d in library_paths() for x in ("-L" + d,)] + ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    tmp = BIND_LIB + ".tmp.%d" % os.getpid()
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), *inc, BIND_SRC, "-o", tmp, *libs],
                   check=True)
    os.replace(tmp, BIND_LIB)
    return BIND_LIB


def build_synth() -> str:
    """Compiles the device-side input generator into libmoda_synth.so."""
    tmp = SYNTH_LIB + ".tmp.%d" % os.getpid()
    subprocess.run([HIPCC, *FLAGS, "-shared", SYNTH_SRC, "-o", tmp], check=True,
                   stderr=subprocess.PIPE if os.environ.get("MODA_QUIET_BUILD") else None)
    os.replace(tmp, SYNTH_LIB)
    return SYNTH_LIB


if __name__ == "__main__":
    print(build_libmoda())
