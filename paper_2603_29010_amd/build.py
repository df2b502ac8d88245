"""Build libucl.so: every HIP translation unit compiled for gfx950 with hipcc, in parallel, in-tree.

Run as ``python -m paper_2603_29010_amd.build`` (or call ``build()``).  Object files and the
library stay inside the package directory; nothing is installed.
"""
import concurrent.futures
import glob
import os
import re
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libucl.so")
# Extension module: the launching entry points as Python calls them (named for the interpreter it is built for: another one does not load it)
CALLS = os.path.join(HERE, "_calls" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CC = os.environ.get("CC", "gcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-disable-promote-alloca-to-lds",
         "-Wno-pass-failed", "-Wno-unused-variable", "-Wno-unused-but-set-variable"]


def _compile(src, force):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    deps = [src] + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(HERE, "..", "include", "ucl.h")]
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(d) for d in deps):
        return obj, ""
    cmd = [HIPCC] + FLAGS + ["-save-temps=obj", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True, cwd=OBJ)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    _check_asm(obj)
    return obj, err


def _check_asm(obj):
    """Refuse kernels that spill to scratch: accumulators must live in registers."""
    stem = os.path.basename(obj)[:-len(".hip.o")]
    for asm in glob.glob(os.path.join(OBJ, stem + "-hip-amdgcn-amd-amdhsa-gfx950.s")):
        text = open(asm).read()
        names = re.findall(r"\.amdhsa_kernel\s+(\S+)", text)
        sizes = re.findall(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", text)
        if len(names) != len(sizes):
            raise RuntimeError(f"{asm}: cannot match kernels to their scratch sizes")
        for name, scratch in zip(names, sizes):
            if int(scratch) != 0:
                raise RuntimeError(f"kernel {name} uses {scratch} bytes of scratch memory")
        if re.search(r"s_swappc_b64", text):
            raise RuntimeError(f"{asm}: a kernel calls a function (a loop body was not inlined)")
        # A buffer resource that the register allocator moved into vector registers (the tile kernels sit at their
        # scalar-register budget) makes every global -> LDS copy a readfirstlane loop: 14 % slower when it happened.
        lines = text.split("\n")
        for k, line in enumerate(lines):
            if "buffer_load_dword" in line and line.rstrip().endswith(" lds") and \
                    any("v_readfirstlane_b32" in x for x in lines[max(0, k - 10):k]) and \
                    any("s_cbranch_execnz" in x for x in lines[k + 1:k + 6]):
                raise RuntimeError(f"{asm}: line {k + 1}: a global -> LDS copy sits in a readfirstlane loop "
                                   "(its buffer resource is held in vector registers)")
        bad = overwritten_store(lines)
        if bad:
            raise RuntimeError(f"{asm}: line {bad[0]}: `{bad[1]}` overwrites data that the store before it may still be reading")
        bad = early_use_of_transpose_reads(lines)
        if bad:
            raise RuntimeError(f"{asm}: line {bad[0]}: `{bad[1]}` touches the result of a transpose read that may still be in flight")


STORE_WAIT_STATES = 2             # between a store of more than 64 bits and a write to its data (what the compiler keeps for stores without a scalar offset)


def overwritten_store(lines):
    """The first (line number, instruction) that overwrites the data of a store of more than 64 bits within STORE_WAIT_STATES behind it, or None: the
    store may still be reading them, also where its offset is in a scalar register and the compiler expects no hazard.  An instruction is one
    wait state, `s_nop n` n + 1; branches are followed to their labels."""
    code, labels = [], {}                             # (line number, instruction, op), and where labels point in it
    for number, line in enumerate(lines, 1):
        ins = line.split(";")[0].strip()
        if ins.endswith(":"):
            labels[ins[:-1]] = len(code)
        elif ins and not ins.startswith("."):
            code.append((number, ins, ins.split()[0]))

    def behind(at, data, left):
        """The same for one store, from instruction `at` with `left` wait states to go."""
        while at < len(code) and left > 0:
            number, ins, op = code[at]
            operands = ins[len(op):].split(",")
            if op.startswith("v_") and _vregs(",".join(operands[:2 if op.startswith("v_swap") else 1])) & data:
                return number, ins
            left -= int(operands[0], 0) + 1 if op == "s_nop" else 1
            if op == "s_branch" or op.startswith("s_cbranch"):
                bad = behind(labels.get(operands[0].strip(), len(code)), data, left)
                if bad:
                    return bad
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                return None
            at += 1
        return None

    for at, (_, ins, op) in enumerate(code):
        m = re.match(r"(buffer|global|flat)_store_dwordx[34]", op)
        if m:
            bad = behind(at + 1, _vregs(ins[len(op):].split(",")[0 if m.group(1) == "buffer" else 1]), STORE_WAIT_STATES)
            if bad:
                return bad
    return None


def _vregs(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        first, last = (m.group(2), m.group(3)) if m.group(2) else (m.group(4), m.group(4))
        out |= {(m.group(1), i) for i in range(int(first), int(last) + 1)}
    return out


def early_use_of_transpose_reads(lines):
    """The kernels' transpose reads are asm statements, for which the compiler counts no waits: the first (line number, instruction)
    that touches the destination of one before a wait covers it, or None.  LDS accesses return in order; lines are taken
    as they stand (a loop's back edge is not followed)."""
    pending = []                                      # destinations of the LDS accesses in flight, oldest first
    for number, line in enumerate(lines, 1):
        ins = line.split(";")[0].strip()
        if not ins or ins.startswith("."):
            continue
        if ins.endswith(":"):
            if ins.startswith("_Z"):
                pending = []
            continue
        op = ins.split()[0]
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", ins)
            if m:
                keep = int(m.group(1))
                pending = pending[len(pending) - keep:] if 0 < keep < len(pending) else pending if keep else []
            elif re.fullmatch(r"s_waitcnt\s+0", ins):
                pending = []
            continue
        if any(pending):
            used = _vregs(ins[len(op):])
            if any(used & dst for dst in pending):
                return number, ins
        if op == "ds_read_b64_tr_b16":
            pending.append(_vregs(ins[len(op):].split(",")[0]))
        elif op.startswith("ds_") or op.startswith("s_load"):
            pending.append(set())
    return None


def _build_calls(force):
    """Without a compiler or Python.h the binding goes through ctypes alone: a warning, and no module of an earlier source is left behind."""
    src, deps = os.path.join(CSRC, "py_calls.c"), [os.path.join(CSRC, "py_calls.c"), os.path.join(HERE, "..", "include", "ucl.h")]
    if not force and os.path.exists(CALLS) and os.path.getmtime(CALLS) >= max(os.path.getmtime(d) for d in deps):
        return
    for stale in (CALLS, os.path.join(os.path.dirname(CALLS), "_calls.so")):         # (the name that every interpreter loads)
        if os.path.exists(stale):
            os.remove(stale)
    cmd = [CC, "-O2", "-Wall", "-Wextra", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], src, "-o", CALLS]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        why = (r.stderr or f"exit status {r.returncode}") if r.returncode else ""
    except OSError as e:
        why = str(e)
    if why:
        warnings.warn(f"the extension module of the launching entry points was not built, calls go through ctypes: {why.strip()[:500]}")


def build(force=False, jobs=None, verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    _build_calls(force)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = jobs or min(8, os.cpu_count() or 1)
    objs = []
    with concurrent.futures.ThreadPoolExecutor(jobs) as ex:
        for obj, err in ex.map(lambda s: _compile(s, force), srcs):
            objs.append(obj)
            if verbose and err.strip():
                print(err, file=sys.stderr)
    newest = max(os.path.getmtime(o) for o in objs)
    if force or not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
