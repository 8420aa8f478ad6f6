"""Builds libmcf.so (HIP kernels for gfx950 + the C ABI) in-tree with hipcc.

hipcc cross-compiles without a GPU.  Objects go to _build/ at the repository root (ignored
by git); the shared library is written next to this file so that it travels with the tree.
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(ROOT, "_build", "mcf")
LIB = os.path.join(HERE, "libmcf.so")
TORCH_EXT = os.path.join(HERE, "_mcf_torch.so")   # extension module of the binding: no kernels, links against libmcf.so
TORCH_SRC = "mcf_torch.cpp"

# -packed-fp32-ops is switched off on purpose: hipcc must not form packed fp32 instructions.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")) and f != TORCH_SRC)


def _headers_mtime():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".h", ".hpp"))]
    hs.append(os.path.join(ROOT, "include", "mcf.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src, force, hdr_mtime, extra=()):
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    if (not force and os.path.exists(obj) and os.path.getmtime(obj) >= os.path.getmtime(src)
            and os.path.getmtime(obj) >= hdr_mtime):
        return obj
    cmd = (["hipcc"] + HIPCC_FLAGS + list(extra) + (["-x", "hip"] if src.endswith(".cpp") else [])
           + ["-c", src, "-o", obj])
    r = subprocess.run(cmd, capture_output=True, text=True, cwd=OBJ_DIR)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed on " + src)
    return obj


_KERNEL_RE = re.compile(r"chain_kernelI(DF16_|DF16b)Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELb([01])ELb([01])ELi(\d+)E")


def _spills_in_loops(text, symbol):
    """Whether any spill instruction (scratch_load / scratch_store) of the kernel `symbol` sits
    in a basic block the compiler marks as part of a loop (its comment after the block's label:
    "in Loop: Header=..." or "... Loop Header: Depth=...").  A register parked in scratch before
    the n loop and fetched after it costs a block two instructions; one moved in and out inside
    the loop costs them every trip."""
    start = text.find("\n" + symbol + ":")
    end = text.find(".Lfunc_end", start)
    if start < 0 or end < 0:
        return True
    in_loop = False
    for line in text[start:end].split("\n"):
        if line.startswith(".LBB") or line.startswith("; %bb."):
            in_loop = "Loop Header" in line or "in Loop:" in line
        elif line.lstrip().startswith(";"):
            if "in Loop: Header" in line or "Loop Header: Depth" in line:
                in_loop = True
        elif in_loop and "scratch_" in line.split(";")[0]:
            return True
    return False


def _write_resource_table(path):
    """Registers and scratch bytes of every compiled kernel, read from the assembly the
    compiler leaves beside the objects (-save-temps); the tile picker uses them as the exact
    form of its on-chip memory rule."""
    rows = []
    for f in sorted(os.listdir(OBJ_DIR)):
        if not (f.startswith("inst_") and f.endswith("gfx950.s")):
            continue
        text = open(os.path.join(OBJ_DIR, f)).read()
        for block in text.split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block)
            m = _KERNEL_RE.search(name.group(1)) if name else None
            if not m:
                continue
            vg = int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
            sg = int(re.search(r"\.sgpr_count:\s+(\d+)", block).group(1))
            scratch = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1))
            dt = 0 if m.group(1) == "DF16_" else 1
            in_loop = 1 if scratch and _spills_in_loops(text, name.group(1)) else 0
            rows.append("    {%d, %s, %d, %d, %d, %d}," % (dt, ", ".join(m.group(i) for i in range(2, 12)), vg, sg, scratch, in_loop))
    if not rows:
        raise RuntimeError("no kernel metadata found under " + OBJ_DIR)
    for f in os.listdir(OBJ_DIR):   # the other by-products of -save-temps are large and unused
        if f.endswith((".bc", ".hipi", ".out", ".hipfb", ".resolution.txt", "x86_64-unknown-linux-gnu.s")):
            os.remove(os.path.join(OBJ_DIR, f))
    with open(path, "w") as out:
        out.write("// generated by build.py from the compiler's kernel metadata; do not edit\n")
        out.write("// {dtype, K, L, mb, rg, ns, nj, softmax, b_kcontig, ksplit, P, vgprs, sgprs, scratch_bytes, spills_in_loops}\n")
        out.write("\n".join(rows) + "\n")
    return len(rows)


def _build_torch_ext():
    """The extension module the chain calls of the binding go through (host code only)."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"),
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           os.path.join(CSRC, TORCH_SRC), "-o", TORCH_EXT, LIB, "-L", os.path.join(t, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_hip", "-ltorch", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True, cwd=HERE)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("build of " + TORCH_EXT + " failed")
    return TORCH_EXT


def build_library(force=True, jobs=8, verbose=False):
    """Compile every source and link libmcf.so.  force=False reuses up-to-date objects."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    hdr = _headers_mtime()
    srcs = sources()
    kernels = [s for s in srcs if s.endswith(".hip")]
    host = [s for s in srcs if not s.endswith(".hip")]
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, force, hdr, ["-save-temps=obj"]), kernels))
    n = _write_resource_table(os.path.join(OBJ_DIR, "mcf_resources.inc"))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs += list(ex.map(lambda s: _compile(s, True, hdr, ["-I", OBJ_DIR]), host))
    if verbose:
        print("kernel resource table:", n, "kernels")
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libmcf.so", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libmcf.so failed")
    _build_torch_ext()
    if verbose:
        print("built", LIB, "from", len(objs), "objects, and", TORCH_EXT)
    return LIB


if __name__ == "__main__":
    build_library(force="--force" in sys.argv, verbose=True)
