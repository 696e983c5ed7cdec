"""Build libflashrnn.so (HIP, gfx950) and the Python binding's native part (g++) in-tree.  `python -m paper_2412_07752_amd.build [--force]`.

Every translation unit is compiled with hipcc for gfx950 only, with the packed-FP32 VALU
instructions disabled (compiler flag, device side).  Objects land in csrc/_build (git-ignored), the
library next to the Python binding.
"""
import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OUT = os.path.join(HERE, "libflashrnn.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -amdgpu-mfma-vgpr-form: MFMA results go to ordinary VGPRs.  Left to itself the compiler puts the accumulators of kernels with
# few waves into AGPRs and copies every result out again (16 moves per time step in the small tile kernels), and the kernels that
# hold R in all 512 registers spill less with it.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-mfma-vgpr-form", "-I", INCLUDE, "-I", CSRC]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _newest_header():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")] + [os.path.join(INCLUDE, "flashrnn.h")]
    return max(os.path.getmtime(h) for h in hs)


def _compile(src, obj, extra=()):
    r = subprocess.run([HIPCC] + FLAGS + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    log = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{log}")
    return log


def binding_stamp():
    """What the native module reads objects and tensors through: the headers of one Python and one torch.  Compiled into it, and compared when it is loaded."""
    import torch
    return f"python {sys.version_info[0]}.{sys.version_info[1]}, torch {torch.__version__} {torch.version.git_version}"


def build_binding(force=False):
    """_flashrnn_binding<ABI tag>.so: the native part of api.py's forward calls (host code, against the running Python and its torch)."""
    import torch
    root, src, name = os.path.dirname(torch.__file__), os.path.join(CSRC, "flashrnn_binding.cpp"), "_flashrnn_binding"
    out = os.path.join(HERE, name + sysconfig.get_config_var("EXT_SUFFIX"))
    if os.path.exists(os.path.join(HERE, name + ".so")):   # (without a tag any Python would load it)
        os.remove(os.path.join(HERE, name + ".so"))
    if not force and os.path.exists(out) and os.path.getmtime(out) >= max(os.path.getmtime(src), os.path.getmtime(os.path.join(INCLUDE, "flashrnn.h"))):
        with open(out, "rb") as f:
            if binding_stamp().encode() + b"\0" in f.read():
                return out
    if os.path.exists(out):   # (nothing old stays where the new one does not compile)
        os.remove(out)
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DFLASHRNN_BUILT_FOR="{binding_stamp()}"',
           "-I", INCLUDE, "-I", sysconfig.get_paths()["include"], "-I", os.path.join(root, "include"), "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"), src, "-o", out, "-L", os.path.join(root, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on flashrnn_binding.cpp:\n{r.stdout}")
    return out


def build(force=False, jobs=None, trace=False):
    """trace=True: the same sources with -DFLASHRNN_TRACE (per-phase clock stamps in the split-group kernels), as
    libflashrnn_trace.so; a measurement build, never what the tests or the benchmark's numbers run on."""
    bdir = os.path.join(CSRC, "_build_trace" if trace else "_build")
    flags_extra = ["-DFLASHRNN_TRACE"] if trace else []
    out = OUT.replace("libflashrnn.so", "libflashrnn_trace.so") if trace else OUT
    os.makedirs(bdir, exist_ok=True)
    hdr = _newest_header()
    todo, objs = [], []
    for src in sources():
        obj = os.path.join(bdir, src[:-4] + ".o")
        objs.append(obj)
        if force or not os.path.exists(obj) or os.path.getmtime(obj) < max(hdr, os.path.getmtime(os.path.join(CSRC, src))):
            todo.append((src, obj))
    jobs = jobs or min(8, os.cpu_count() or 1)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        binding = ex.submit(build_binding, force)
        for log in ex.map(lambda so: _compile(*so, extra=flags_extra), todo):
            if log.strip():
                print(log)
    if todo or not os.path.exists(out) or os.path.getmtime(out) < max(map(os.path.getmtime, objs)):
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", out])
    try:   # (the library is whole without it: a machine that has hipcc alone builds and uses the C ABI)
        binding.result()
    except Exception as e:
        warnings.warn(f"the native part of the Python binding was not built, forward calls take a few microseconds more through ctypes: {e}", RuntimeWarning)
    return out


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, trace="--trace" in sys.argv))
