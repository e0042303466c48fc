"""Build libmxp.so (the C-ABI HIP library) for gfx950 with hipcc, in-tree."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmxp.so")
PROBE_DIR = os.path.join(HERE, "probe")
PROBE_LIB = os.path.join(PROBE_DIR, "libmxp_probe.so")      # bench-only measurement aid, not part of the product ABI
BINDING_SRC = os.path.join(CSRC, "mxp_binding.cpp")
BINDING_LIB = os.path.join(HERE, "_mxp_binding.so")         # host side of the binding's frequent calls (a Python module)
SOURCES = ["mxp_quantize.hip", "mxp_convert.hip", "mxp_gemm.hip", "mxp_w4a16.hip", "mxp_bf16.hip", "mxp_wide.hip", "mxp_canon.hip", "mxp_few_rows.hip"]
HEADERS = [os.path.join(CSRC, "mxp_common.h"), os.path.join(CSRC, "mxp_decode.h"), os.path.join(CSRC, "mxp_tile.h"), os.path.join(CSRC, "mxp_prepack_body.h"), os.path.join(ROOT, "include", "mxp.h")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    return "hipcc"


def _binding_command():
    import sysconfig
    import torch
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include",
           sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DMXP_TORCH_VERSION="%s"' % torch.__version__] +
            ["-I" + d for d in inc] +
            [BINDING_SRC, "-o", BINDING_LIB, "-L" + os.path.join(t, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-ltorch"])


def _newer(target, deps):
    return os.path.exists(target) and all(os.path.getmtime(d) <= os.path.getmtime(target) for d in deps)


def up_to_date():
    """The libraries and the binding's native part, the latter also against torch."""
    import torch
    torch_version = os.path.join(os.path.dirname(torch.__file__), "version.py")
    return (_newer(LIB, [os.path.join(CSRC, s) for s in SOURCES] + HEADERS + [os.path.abspath(__file__)]) and
            _newer(PROBE_LIB, [os.path.join(PROBE_DIR, f) for f in ("mxp_probe.hip", "mxp_probe.h")] + HEADERS) and
            _newer(BINDING_LIB, [BINDING_SRC, HEADERS[-1], torch_version]))


def build_binding():
    """Compile the binding's native part.  The package works without it, with more host time per call: a machine that cannot compile it
    (no host compiler, no headers of torch or Python) gets a warning, and no file that another torch left."""
    import warnings
    if os.path.exists(BINDING_LIB):
        os.remove(BINDING_LIB)
    try:
        p = subprocess.run(_binding_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        failed, why = p.returncode != 0, p.stdout
    except OSError as e:
        failed, why = True, str(e)
    if failed:
        warnings.warn("_mxp_binding.so was not built, calls will take the slower general code:\n" + why, RuntimeWarning)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and up_to_date():
        return LIB
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for s in SOURCES:
        o = os.path.join(objdir, s.replace(".hip", ".o"))
        objs.append(o)
        cmd = [_hipcc()] + FLAGS + ["-c", os.path.join(CSRC, s), "-o", o]
        if verbose:
            print(" ".join(cmd))
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    pcmd = [_hipcc()] + FLAGS + ["-I" + PROBE_DIR, "-shared", os.path.join(PROBE_DIR, "mxp_probe.hip"), "-o", PROBE_LIB]
    procs.append(("mxp_probe.hip", subprocess.Popen(pcmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    build_binding()                                          # (beside the compilations above)
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (s, out))
        if out.strip() and verbose:
            print(out)
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
