"""Build libllmq.so (the gfx950 kernels and their C ABI) in-tree with hipcc, and the Python module over it with g++.  The library needs
nothing but hipcc: where the module does not build, the library is there without it (and llmq.py takes the ctypes path)."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libllmq.so")
BINDING = os.path.join(HERE, "_binding.so")       # the Python module of csrc/binding.cpp
# gemm_tiles_*.hip: the tile kernels of one operand-kind pair and layout each (all tile shapes), so that they compile
# side by side; the largest come first.
TILE_SOURCES = ["gemm_tiles_e4m3_e4m3.hip", "gemm_tiles_e5m2_e4m3.hip", "gemm_tiles_e4m3_e5m2.hip", "gemm_tiles_e5m2_e5m2.hip",
                "gemm_tiles_e4m3_e4m3_abt.hip", "gemm_tiles_e4m3_e4m3_bt.hip", "gemm_tiles_e4m3_e4m3_at.hip",
                "gemm_tiles_e5m2_e4m3_abt.hip", "gemm_tiles_e5m2_e4m3_bt.hip", "gemm_tiles_e5m2_e4m3_at.hip",
                "gemm_tiles_bf16_bf16.hip"]
# the same for ragged shapes
TILE_SOURCES += ["gemm_edge_%s.hip" % kind for kind in
                 ("e4m3_e4m3", "e5m2_e4m3", "e4m3_e5m2", "e5m2_e5m2", "bf16_bf16",
                  "e4m3_e4m3_bt", "e5m2_e4m3_bt", "e4m3_e4m3_abt", "e5m2_e4m3_abt")]
SOURCES = TILE_SOURCES + ["gemm.hip", "gemm_tmajor.hip", "api.hip", "amax.hip", "quantize.hip", "swiglu.hip", "rmsnorm.hip", "calibrate.hip"]
# Sources that hold tile kernels (see check_accumulator_reads).
CHECKED_SOURCES = set(TILE_SOURCES) | {"gemm.hip"}
# packed-fp32 VALU ops are disabled on purpose (they have produced silent wrong results on this
# hardware pool); never add -ffast-math: the scale needs a correctly rounded division.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _registers(line: str):
    """The vector and accumulator registers an instruction names, as (file, number)."""
    found = {(f, int(n)) for f, n in re.findall(r"\b([av])(\d+)\b", line)}
    for f, lo, hi in re.findall(r"\b([av])\[(\d+):(\d+)\]", line):
        found.update((f, n) for n in range(int(lo), int(hi) + 1))
    return found


def check_accumulator_reads(src: str, asm: str) -> None:
    """The tile kernels write their MFMAs out as inline assembly, so the compiler does not know that an
    accumulator read must keep its distance from the MFMA that wrote it.  The kernels' own code keeps it: nothing
    but MFMAs touches the registers MFMAs write (accumulator registers, and in the largest tiles ordinary ones too) from the
    first MFMA to the wait states behind the K loop (`s_nop 15`).  Code the register allocator adds on its own (copies between
    the register files, spills of accumulators) would not, so any such instruction in that stretch of the generated assembly is
    a build error.  Allowed is the zeroing of the accumulators, which may be repeated on the path of a single K step, behind the K
    loop in the text: writes of an ordinary register to the accumulator file, and, in a block without MFMAs that only code in
    front of the first MFMA jumps to, to the ordinary registers among the accumulators."""
    bad = []
    checked = 0
    for m in re.finditer(r"^(_ZN4llmq16gemm_tile_kernel\w*):[^\n]*\n(.*?)^\.Lfunc_end", asm, re.S | re.M):
        name, body = m.group(1), m.group(2)
        code = [l.split(";")[0].strip() for l in body.splitlines()]
        code = [l for l in code if l and (not l.startswith(".") or l.startswith(".LBB")) and (not l.endswith(":") or l.startswith(".LBB"))]
        mfma = [i for i, l in enumerate(code) if l.startswith("v_mfma_")]
        if not mfma:
            continue                                  # the kernel that only adds up pieces
        checked += 1
        drain = next((i for i in range(mfma[-1], len(code)) if code[i] == "s_nop 15"), None)
        if drain is None:
            bad.append("%s: no wait states behind the last MFMA" % name)
            continue
        accumulators = {("a", n) for n in range(256)}
        for i in mfma:
            accumulators |= _registers(code[i].split()[1])
        label_at = {l[:-1]: i for i, l in enumerate(code) if l.endswith(":")}
        jumps = [(i, label_at[l.split()[-1]]) for i, l in enumerate(code) if re.match(r"s_c?branch", l) and l.split()[-1] in label_at]
        zeroing, end = set(), mfma[0]                 # lines of blocks that may zero accumulators
        for i in range(mfma[0], drain):
            if not code[i].endswith(":") or not re.match(r"s_branch|s_endpgm", code[i - 1]):
                continue
            end = next((k for k in range(i + 1, drain) if code[k].endswith(":") or re.match(r"s_c?branch", code[k])), drain)
            if all(k < mfma[0] for k, to in jumps if to == i) and not any(i < k < end for k in mfma):
                zeroing.update(range(i, end))
        for i in range(mfma[0], drain):
            l = code[i]
            if l.startswith("v_mfma_") or l.endswith(":") or not (_registers(l) & accumulators):
                continue
            if re.fullmatch(r"v_accvgpr_write_b32 a\d+, v\d+", l) and (i in zeroing or ("v", int(l.split("v")[-1])) not in accumulators):
                continue
            if i in zeroing and re.match(r"v_mov_b(32|64)_e32 ", l):
                continue
            bad.append("%s: %s" % (name, l))
            break
    if not checked:
        raise RuntimeError("%s: no tile kernel found in the generated assembly" % src)
    if bad:
        raise RuntimeError("%s: accumulator registers touched inside the MFMA stretch:\n  %s" % (src, "\n  ".join(bad)))


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    work = tempfile.mkdtemp(prefix="llmq_build_")
    try:
        return _build_in(work, hipcc, verbose)
    finally:
        shutil.rmtree(work, ignore_errors=True)


def binding_commands(obj: str, lib_dir: str, out: str):
    """Compile and link commands of the Python module (CPU code; the library is found beside it at run time)."""
    import torch
    root = os.path.dirname(torch.__file__)
    includes = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]]
    cxx = os.environ.get("CXX", "g++")
    abi = "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)
    return ([cxx, "-O2", "-std=c++17", "-fPIC", "-Wall", abi] + [a for i in includes for a in ("-isystem", i)] + ["-c", os.path.join(CSRC, "binding.cpp"), "-o", obj],
            [cxx, "-shared", obj, "-o", out, "-L", lib_dir, "-lllmq", "-Wl,-rpath,$ORIGIN", "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"])


def _run_binding(command):
    """A command of the module's build as a process, or None with a message where it cannot even start."""
    try:
        return subprocess.Popen(command, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except OSError as e:
        print("%s: %s" % (command[0], e), file=sys.stderr)
        return None


def _finish_binding(process) -> bool:
    if process is None:
        return False
    out, _ = process.communicate()
    if process.returncode != 0:
        print(out, file=sys.stderr)
    return process.returncode == 0


def _build_in(work: str, hipcc: str, verbose: bool) -> str:
    objs = []
    procs = []
    new_lib, new_binding = os.path.join(work, "libllmq.so"), os.path.join(work, "_binding.so")
    compile_binding = link_binding = binding = None
    try:
        compile_binding, link_binding = binding_commands(os.path.join(work, "binding.o"), work, new_binding)
    except ImportError as e:                          # no PyTorch here
        print("binding.cpp: %s" % e, file=sys.stderr)
    if compile_binding:
        binding = _run_binding(compile_binding)
    for src in SOURCES:
        obj = os.path.join(work, src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if src in CHECKED_SOURCES:
            cmd.append("-save-temps=obj")             # keeps the device assembly next to the object
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            print("FAILED: %s\n%s" % (src, out), file=sys.stderr)
        elif verbose and out.strip():
            print(out)
    binding_built = _finish_binding(binding)
    if failed:
        raise RuntimeError("hipcc failed")
    for src in sorted(CHECKED_SOURCES):
        with open(os.path.join(work, src.replace(".hip", "-hip-amdgcn-amd-amdhsa-gfx950.s"))) as f:
            check_accumulator_reads(src, f.read())
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", new_lib])
    binding_built = binding_built and _finish_binding(_run_binding(link_binding))
    # Both are there (or the module is not going to be): now they replace the old ones.  A module of another build must not stay
    # beside the new library.
    if os.path.exists(BINDING):
        os.remove(BINDING)
    _replace(new_lib, LIB)
    if binding_built:
        _replace(new_binding, BINDING)
    else:
        print("FAILED: binding.cpp: the calls of llmq.py take the ctypes path", file=sys.stderr)
    return LIB


def _replace(new: str, path: str) -> None:
    tmp = path + ".tmp.%d" % os.getpid()
    shutil.copy(new, tmp)
    os.replace(tmp, path)


if __name__ == "__main__":
    print(build(verbose=True))
