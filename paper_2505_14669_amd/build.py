"""Build the HIP library (paper_2505_14669_amd/libquartet.so) for gfx950 with hipcc and, on top of it, the autograd node of
the torch layer (paper_2505_14669_amd/_nn_native.<Python's tag>.so) with g++."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libquartet.so")
NN_LIB = os.path.join(HERE, "_nn_native" + sysconfig.get_config_var("EXT_SUFFIX"))     # another Python does not take it for its own
OBJDIR = os.path.join(HERE, "_build")
SOURCES = ["api.hip", "quant_kernels.hip", "gemm_kernels.hip", "gemm_split_kernels.hip", "epilogue_kernels.hip", "fp8_kernels.hip", "probe_kernels.hip"]

# -ffp-contract=off: the Hadamard butterflies and scale arithmetic must not be fused into FMAs;
# packed-fp32 VALU ops are disabled (they have given wrong results on these machines).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


def _compile(src):
    obj = os.path.join(OBJDIR, src.replace(".hip", ".o"))
    cmd = ["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    return obj, out


def _compile_nn():
    """nn_autograd.cpp -> object file: host code against the installed torch's headers."""
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(OBJDIR, "nn_autograd.o")
    dirs = include_paths(device_type="cuda") + ["/opt/rocm/include", sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for d in dirs:
        cmd += ["-isystem", d]
    r = subprocess.run(cmd + ["-c", os.path.join(CSRC, "nn_autograd.cpp"), "-o", obj], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on nn_autograd.cpp:\n{r.stdout}")
    return obj, os.path.join(os.path.dirname(torch.__file__), "lib")


def _have_torch():
    try:
        import torch  # noqa: F401
    except ImportError:
        return False
    return True


def build(verbose=False):
    """Returns the library's path.  The library needs hipcc alone and is linked whatever becomes of the torch node; without torch, which
    the node's only user imports as well, there is no node."""
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=5) as ex:
        nn = ex.submit(_compile_nn) if _have_torch() else None
        results = list(ex.map(_compile, SOURCES))
    if verbose:
        for _, out in results:
            if out.strip():
                print(out)
    objs = [o for o, _ in results]
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    if nn is not None:
        nn_obj, torch_lib = nn.result()
        # the torch libraries are in the process already when this is imported; libquartet.so lies beside it
        subprocess.run(["g++", "-shared", "-o", NN_LIB, nn_obj, "-L" + HERE, "-l:libquartet.so", "-L" + torch_lib, "-ltorch_python",
                        "-ltorch_cpu", "-ltorch_hip", "-lc10_hip", "-lc10", "-Wl,-rpath,$ORIGIN"], check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
