"""Build libwmdec.so (HIP, gfx950 only) in-tree with hipcc, and the native Python binding with g++."""
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig
import tempfile

if __package__:
    from . import asm_check
else:
    import asm_check

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libwmdec.so")
BINDING = os.path.join(HERE, "_binding.so")

SOURCES = ["api.cpp", "kernels_gn.hip", "kernels_conv_direct.hip", "kernels_conv_mfma.hip", "kernels_conv_rows.hip", "kernels_conv_rows_bf16.hip", "kernels_conv_ksplit.hip", "kernels_conv_up.hip",
           "kernels_conv_taps.hip", "kernels_misc.hip", "kernels_attn.hip", "kernels_adaln.hip"]

# what asm_check looks for beside the stores of every source: kernels with matrix instructions in inline assembly, kernels that must not spill
CHECKED = {"kernels_attn.hip": {"scores": "flash_attn_kernel"}, "kernels_conv_rows.hip": {"spills": "conv_mfma_kernel"},
           "kernels_conv_rows_bf16.hip": {"spills": "conv_mfma_kernel"}}

# sources that include another one
INCLUDES = {"kernels_conv_rows_bf16.hip": "kernels_conv_rows.hip"}

FLAGS = ["-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes"]


def _headers_mtime():
    m = 0.0
    for root in (CSRC, os.path.join(os.path.dirname(HERE), "include")):
        for f in os.listdir(root):
            if f.endswith((".hpp", ".h")):
                m = max(m, os.path.getmtime(os.path.join(root, f)))
    return m


def device_assembly(src):
    """The device assembly that the flags of the build make of a source file."""
    r = subprocess.run(["hipcc"] + FLAGS + ["-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", "-"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr))
    return r.stdout


def _compile(src, force):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(path), os.path.getmtime(os.path.join(CSRC, INCLUDES.get(src, src))), _headers_mtime()):
        return obj
    with tempfile.TemporaryDirectory() as temps:   # the device assembly on its way into the object
        cmd = ["hipcc"] + FLAGS + ["-save-temps", "-c", path, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True, cwd=temps)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
        if out.strip():
            sys.stderr.write(out + "\n")
        assembly = glob.glob(os.path.join(temps, "*amdgcn*.s"))
        if len(assembly) != 1:
            os.remove(obj)
            raise RuntimeError("%s: %d device assembly files" % (src, len(assembly)))
        with open(assembly[0]) as f:
            faults = asm_check.check_source(f.read(), **CHECKED.get(src, {}))
    if faults:
        os.remove(obj)
        raise RuntimeError("%s: the compiled code breaks what its source relies on:\n%s" % (src, "\n".join(faults)))
    return obj


def build_binding(force=True):
    """The native Python module (csrc/binding.cpp) against the installed torch."""
    src = os.path.join(CSRC, "binding.cpp")
    if not force and os.path.exists(BINDING) and os.path.getmtime(BINDING) >= max(os.path.getmtime(src), _headers_mtime()):
        return BINDING
    import torch
    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), src, "-o", BINDING]
    cmd += ["-I" + d for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]]
    cmd += ["-L" + d for d in cpp_extension.library_paths()] + ["-lc10", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for binding.cpp:\n%s" % r.stderr)
    return BINDING


def build(force=True, jobs=8):
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        binding = ex.submit(build_binding, force)
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
        binding.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    return LIB


def build_diag():
    """The stand-alone diagnostic that measures what the matrix pipe sustains on this machine."""
    exe = os.path.join(HERE, "mfma_ceiling")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           os.path.join(CSRC, "diag", "mfma_ceiling.hip"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    return exe


if __name__ == "__main__":
    if "--diag" in sys.argv:
        print(build_diag())
    else:
        print(build(force="--incremental" not in sys.argv))
