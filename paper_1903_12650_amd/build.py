"""Compile the HIP sources under csrc/ for gfx950 into librn50_hip.so, and the native part of the Python binding into _ops.so
(both in-tree)."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librn50_hip.so")
OPS_SRC, OPS = os.path.join(CSRC, "python", "ops.cpp"), os.path.join(HERE, "_ops.so")
OBJ_DIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed-FP32 instructions are switched off for every device compile.
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # keep MFMA accumulators in ordinary VGPRs: no AGPR<->VGPR copies around the main loops
         "-mllvm", "-amdgpu-mfma-vgpr-form"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


# Tuning builds (RN50_TUNING=1 in the environment of this script) compile in the environment-variable overrides of
# tile shapes that the sweeps use; the product build has none.
if os.environ.get("RN50_TUNING") == "1":
    FLAGS.append("-DRN50_TUNING")


def _compile(src, force):
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    deps = [src] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    deps.append(os.path.join(HERE, "..", "include", "rn50_hip.h"))
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    cmd = [HIPCC] + FLAGS + (["-x", "hip"] if src.endswith(".hip") else []) + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr[-8000:]))
    warn = [l for l in r.stderr.splitlines() if "warning" in l and "packed-fp32-ops" not in l]
    if warn:
        sys.stderr.write("\n".join(warn[:20]) + "\n")
    return obj


def _compile_ops(force):
    """The native marshalling of the per-layer Python calls: an object now (host code against torch's headers), linked below."""
    import sysconfig
    from torch.utils import cpp_extension
    obj = os.path.join(OBJ_DIR, "ops.cpp.o")
    deps = [OPS_SRC, os.path.join(HERE, "..", "include", "rn50_hip.h")]
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    inc = [a for p in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]] for a in ("-isystem", p)]
    subprocess.check_call(["g++", "-O2", "-fPIC", "-std=c++17", "-Wall"] + inc + ["-c", OPS_SRC, "-o", obj])
    return obj


def _link_ops(obj):
    from torch.utils import cpp_extension
    libs = [a for p in cpp_extension.library_paths() for a in ("-L" + p,)]
    subprocess.check_call(["g++", "-shared", "-o", OPS, obj, "-L" + HERE, "-l:librn50_hip.so", "-Wl,-rpath,$ORIGIN"] + libs +
                          ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"])


def build(force=True, jobs=8):
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        ops = ex.submit(_compile_ops, force)
        objs = list(ex.map(lambda s: _compile(s, force), sources()))
    # --no-undefined: a kernel whose host stub was not emitted must fail here, not at load time
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,--no-undefined", "-o", LIB] + objs)
    _link_ops(ops.result())
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
