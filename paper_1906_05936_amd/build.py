"""Builds liblsgd.so (HIP, gfx950) and the binding's extension _marshal (host
code) in-tree next to this file.

Every HIP translation unit is compiled with:
  -ffp-contract=off       no a*b+c contraction into fused multiply-add: each
                          operation of the update is rounded on its own;
  -Xclang -target-feature -Xclang -packed-fp32-ops
                          no packed binary32 instructions (v_pk_*_f32);
  -fvisibility=hidden     only the LSGD_API (extern "C") symbols are exported.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "liblsgd.so")
SOURCES = ["lsgd_plan_pow2_f32.hip", "lsgd_plan_pow2_bf16.hip", "lsgd_flat_pow2_f32.hip", "lsgd_flat_pow2_bf16.hip",
           "lsgd_plan_np2.hip", "lsgd_flat_np2.hip", "lsgd_plan.hip", "lsgd_flat.hip", "lsgd_split.hip", "lsgd_stream.hip",
           "lsgd_common.hip", "lsgd_bench.hip", "lsgd_noalloc.hip"]
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-fvisibility=hidden", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-I" + INCLUDE, "-I" + CSRC,
]


# Every kernel keeps its working set in registers: one that spills to scratch
# memory runs far below the bandwidth bound (a four-unit 16x4 step kernel
# spilled 2.3 KB per lane and ran at half speed). The compiler's per-kernel
# resource remarks are read back and a spilling kernel fails the build.
RESOURCE_REMARKS = ["-Rpass-analysis=kernel-resource-usage"]


def spilling_kernels(remarks: str):
    """(kernel, scratch bytes per lane) for every kernel whose resource-usage
    remark reports scratch memory."""
    import re
    out, name = [], None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name and int(m.group(1)) > 0:
            out.append((name, int(m.group(1))))
    return out


def _compile(src, verbose):
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + CFLAGS + RESOURCE_REMARKS + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s%s" % (src, r.stdout, r.stderr))
    spills = spilling_kernels(r.stderr)
    if spills:
        raise RuntimeError("kernels of %s spill to scratch memory (bytes per lane): %s"
                           % (src, ", ".join("%s %d" % k for k in spills)))
    return obj


# The binding's CPython extension (csrc/marshal.cpp): host code, against the
# headers of the installed torch and Python. Its name carries Python's ABI tag,
# so that another Python does not find it, and it holds torch_build(), which the
# binding compares: torch's tensor layouts are compiled in.
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))


def torch_build() -> str:
    """The torch build that _marshal is compiled against."""
    import torch
    return "%s %s" % (torch.__version__, torch.version.git_version)


def _compile_marshal(verbose):
    import torch
    from torch.utils import cpp_extension
    obj = os.path.join(BUILD_DIR, "marshal.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I" + INCLUDE,
           '-DLSGD_TORCH_BUILD="%s"' % torch_build(), "-I" + CSRC, "-isystem", sysconfig.get_paths()["include"]]
    for d in cpp_extension.include_paths():
        cmd += ["-isystem", d]
    cmd += ["-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on marshal.cpp:\n%s%s" % (r.stdout, r.stderr))
    return obj


def _link_marshal(obj, verbose):
    from torch.utils import cpp_extension
    tmp = MARSHAL + ".tmp%d" % os.getpid()
    cmd = ["g++", "-shared", "-o", tmp, obj, "-L" + PKG, "-l:liblsgd.so", "-Wl,-rpath,$ORIGIN"]
    cmd += ["-L" + d for d in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    subprocess.run(cmd, check=True)
    os.replace(tmp, MARSHAL)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    jobs = min(len(SOURCES) + 1, max(1, min(16, os.cpu_count() or 1)))
    with ThreadPoolExecutor(jobs) as ex:
        marshal = ex.submit(_compile_marshal, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-Wl,--no-undefined", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    _link_marshal(marshal.result(), verbose)
    return LIB


def _code_only(text: str) -> str:
    """Source text without comments and with whitespace runs collapsed, so that
    a comment-only edit keeps the digest (string literals are kept as they are;
    the sources hold no comment markers inside strings)."""
    import re
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def source_digest() -> str:
    """SHA-256 over the kernel sources and public headers (comments and layout
    stripped) and the build flags: identifies the kernels a stored profile was
    taken from."""
    import hashlib
    h = hashlib.sha256()
    h.update(" ".join(CFLAGS).replace(ROOT, "").encode())
    files = sorted(os.listdir(CSRC))
    for name in files:
        if name.endswith((".hip", ".hpp")):
            with open(os.path.join(CSRC, name)) as f:
                h.update(name.encode() + b"\0" + _code_only(f.read()).encode())
    for name in ("lsgd.h", "lsgd_bench.h"):
        with open(os.path.join(INCLUDE, name)) as f:
            h.update(_code_only(f.read()).encode())
    return h.hexdigest()


if __name__ == "__main__":
    print(build(verbose=True))
