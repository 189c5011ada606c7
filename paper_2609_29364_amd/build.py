"""Build libnebulasd.so for gfx950 with hipcc, and the torch marshalling module
(in-tree, no JIT cache)."""
import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_PATH = os.path.join(HERE, "libnebulasd.so")
SOURCES = ["status.cpp", "kv_gather.hip", "verify_attention.hip", "spec_accept.hip",
           "copy_plan.cpp", "kv_commit.hip", "scheduler.cpp", "check_plan.cpp"]
# bandwidth probes for the measurement of practical ceilings: a library of their own
PROBE_SOURCES = ["hbm_probe.hip"]
PROBE_LIB_PATH = os.path.join(HERE, "libnsd_probe.so")
# the torch marshalling module (host code)
BINDING_SOURCE = "torch_binding.cpp"
BINDING_PATH = os.path.join(HERE, "_nsd_torch.so")
ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
          # packed fp32 VALU forms stay off: only scalar fp32 instructions are emitted
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wall", "-Wno-unused-function", f"-I{os.path.join(ROOT, 'include')}"]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC] + CFLAGS + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def _link(objs, path):
    tmp = path + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, path)


def _rocm_include():
    """The include folder with HIP's headers: ROCM_PATH's, the one beside HIPCC (a bare name is
    looked up in PATH, links are followed), or the default installation's."""
    roots = [os.environ.get("ROCM_PATH")]
    hipcc = shutil.which(HIPCC)
    for path in (hipcc, hipcc and os.path.realpath(hipcc)):
        roots.append(path and os.path.dirname(os.path.dirname(path)))
    for root in filter(None, roots + ["/opt/rocm"]):
        if os.path.exists(os.path.join(root, "include", "hip", "hip_runtime_api.h")):
            return os.path.join(root, "include")
    raise RuntimeError(f"HIP's headers are not beside {HIPCC} nor under ROCM_PATH")


def _build_binding():
    """The marshalling module; without a host compiler or torch's headers none is built (the
    package then submits through ctypes), and one of other sources does not stay."""
    torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
    cxx = os.environ.get("CXX", "g++")
    headers = os.path.join(torch_dir, "include", "torch", "csrc", "autograd", "python_variable.h")
    if not shutil.which(cxx) or not os.path.exists(headers):
        print(f"no {BINDING_SOURCE} built: {cxx} or torch's headers are missing", file=sys.stderr)
        if os.path.exists(BINDING_PATH):
            os.remove(BINDING_PATH)
        return
    tmp = BINDING_PATH + ".tmp"
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-I{os.path.join(ROOT, 'include')}",
           "-isystem", os.path.join(torch_dir, "include"),
           "-isystem", os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
           "-isystem", _rocm_include(),
           f"-I{sysconfig.get_paths()['include']}", os.path.join(CSRC, BINDING_SOURCE),
           "-o", tmp, f"-L{os.path.join(torch_dir, 'lib')}", "-ltorch_python", "-ltorch",
           "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {BINDING_SOURCE} failed:\n{r.stderr}")
    os.replace(tmp, BINDING_PATH)


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared libraries (the round's library,
    the bandwidth probes and the torch marshalling module); returns the round
    library's path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = SOURCES + PROBE_SOURCES
    with ThreadPoolExecutor(max_workers=min(4, len(srcs))) as ex:
        binding = ex.submit(_build_binding)
        objs = dict(zip(srcs, ex.map(_compile, srcs)))
        binding.result()
    _link([objs[s] for s in SOURCES], LIB_PATH)
    _link([objs[s] for s in PROBE_SOURCES], PROBE_LIB_PATH)
    if verbose:
        print(f"built {LIB_PATH} and {PROBE_LIB_PATH}", file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
