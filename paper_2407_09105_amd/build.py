"""Build the HIP libraries (gfx950) in-tree with hipcc: libvarlen_attn.so, the attention library
(csrc/*.hip), and libva_probes.so, the benchmark's measurement aids (probes/*.hip); and with g++ the C++ part of
the Python binding, _va_native (native/va_native.cpp), where torch and g++ are there."""
import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
PROBES = os.path.join(HERE, "probes")
LIB = os.path.join(HERE, "libvarlen_attn.so")
PROBES_LIB = os.path.join(HERE, "libva_probes.so")
NATIVE_LIB = os.path.join(HERE, "_va_native" + sysconfig.get_config_var("EXT_SUFFIX"))  # of this interpreter only
OBJ_DIR = os.path.join(HERE, "_build")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]

TARGETS = ((LIB, CSRC), (PROBES_LIB, PROBES))


def sources(src_dir=CSRC):
    return sorted(glob.glob(os.path.join(src_dir, "*.hip")))


def native_command():
    """Command that builds _va_native for the torch that is installed, or None without torch or g++."""
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        return None
    if shutil.which("g++") is None:
        return None
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-I" + os.path.join(ROOT, "include"),
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", f'-DVA_TORCH_VERSION="{torch.__version__}"',
            *["-isystem" + p for p in (*cpp_extension.include_paths(), sysconfig.get_path("include"))],
            os.path.join(HERE, "native", "va_native.cpp"), "-o", NATIVE_LIB,
            *["-L" + p for p in cpp_extension.library_paths()], "-ltorch", "-ltorch_cpu", "-ltorch_python", "-lc10"]


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source and link the shared libraries; always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = {lib: [] for lib, _ in TARGETS}
    cmds = []
    for lib, src_dir in TARGETS:
        for src in sources(src_dir):
            obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
            objs[lib].append(obj)
            cmds.append((lib, [hipcc, *FLAGS, "-I" + src_dir, *extra_flags, "-c", src, "-o", obj]))
    native = native_command()
    if native is None:
        print("no torch or no g++: the Python binding's C++ part is not built", file=sys.stderr)
    else:
        cmds.append((NATIVE_LIB, native))
    procs = []
    for lib, cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((lib, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = set()
    for lib, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines()
                        if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
        if p.returncode != 0:
            failed.add(lib)
            print(out, file=sys.stderr)
        elif verbose and out.strip():
            print(out)
    for lib, _ in TARGETS:  # the C libraries do not need the binding's C++ part
        if not failed - {NATIVE_LIB}:
            subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs[lib], "-o", lib])
    if failed:
        raise RuntimeError("a compiler failed: " + ", ".join(sorted(os.path.basename(lib) for lib in failed)))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
