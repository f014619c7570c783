"""Build libstepq.so in-tree for gfx950.

Each source is compiled on its own (the .hip files with hipcc for gfx950,
the host-only setup code with g++) and the objects are linked by hipcc.
Mixing a `-x c++` source into one hipcc command makes hipcc drop
--offload-arch and fall back to its default target, so the link step is
followed by a check that the library's device bundle is gfx950 and only
gfx950.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libstepq.so")
HIP_SOURCES = ["stepq_host.hip", "stepq_kernels.hip", "stepq_refit.hip", "stepq_rowmax.hip", "stepq_tiles.hip"]
CXX_SOURCES = ["stepq_setup.cpp", "stepq_plan.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

HIP_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms stay off: scalar fp32 only on the device
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core accumulators in ordinary VGPRs: the decode bodies then fit
    # 64 registers (8 waves per SIMD) without a separate AGPR block
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-function",
]
CXX_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-pthread"]
# the binding's native argument checks: a Python module against torch's headers
ARGS_SOURCE = "stepq_args.cpp"
ARGS_MODULE = os.path.join(HERE, "_stepq_args.so")


def device_targets(path: str) -> list[str]:
    """Offload targets named in a built library's device bundle."""
    data = open(path, "rb").read()
    return sorted(set(t.decode() for t in re.findall(rb"hipv4-amdgcn-amd-amdhsa--(gfx[0-9a-f]+)", data)))


def args_command(out: str, csrc: str) -> list[str] | None:
    """The command that builds the binding's native checks, or None without
    Python's and torch's headers (the library needs neither)."""
    try:
        import torch
        from torch.utils.cpp_extension import include_paths
    except ImportError:
        return None
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    py = sysconfig.get_paths()["include"]
    if not (os.path.exists(os.path.join(py, "Python.h"))
            and any(os.path.exists(os.path.join(d, "ATen", "core", "Tensor.h")) for d in include_paths())):
        return None
    inc = [f for d in include_paths() + [py, os.path.join(ROOT, "include")] for f in ("-I", d)]
    return (["g++"] + CXX_FLAGS + ["-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}"] + inc
            + [os.path.join(csrc, ARGS_SOURCE), "-o", out, "-L", tlib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"])


def build(extra_flags: list[str] | None = None, out: str = LIB, verbose: bool = False, csrc: str = CSRC,
          build_dir: str = BUILD_DIR) -> str:
    os.makedirs(build_dir, exist_ok=True)
    objs = []

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, cwd=csrc, stderr=subprocess.PIPE, text=True)
        # hipcc's host pass does not know the device-only feature flag; drop that note
        for line in r.stderr.splitlines():
            if "packed-fp32-ops' is not a recognized feature" not in line:
                print(line, file=sys.stderr)
        if r.returncode != 0:
            raise subprocess.CalledProcessError(r.returncode, cmd)

    inc = ["-I", os.path.join(ROOT, "include"), "-I", csrc]
    cmds = []
    for s in HIP_SOURCES:
        o = os.path.join(build_dir, s + ".o")
        cmds.append([HIPCC] + HIP_FLAGS + (extra_flags or []) + inc + ["-c", os.path.join(csrc, s), "-o", o])
        objs.append(o)
    for s in CXX_SOURCES:
        o = os.path.join(build_dir, s + ".o")
        cmds.append(["g++"] + CXX_FLAGS + inc + ["-c", os.path.join(csrc, s), "-o", o])
        objs.append(o)
    # the module belongs to the package, not to one library: a library of
    # another name is used through it too
    module = args_command(ARGS_MODULE + ".tmp", csrc) if out == LIB or not os.path.exists(ARGS_MODULE) else None
    if module is not None:
        cmds.append(module)
    elif out == LIB:
        print(f"{ARGS_MODULE}: not built (no Python or torch headers); the binding checks arguments in Python",
              file=sys.stderr)
        if os.path.exists(ARGS_MODULE):
            os.remove(ARGS_MODULE)      # of an earlier build, perhaps against another torch
    # the translation units are independent: compile them side by side
    with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as ex:
        for f in [ex.submit(run, c) for c in cmds]:
            f.result()
    out = os.path.abspath(out)
    tmp = out + ".tmp"
    run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-pthread", "-o", tmp] + objs)
    targets = device_targets(tmp)
    if targets != [ARCH]:
        os.remove(tmp)
        raise RuntimeError(f"libstepq device bundle targets {targets}, expected only {ARCH}")
    os.replace(tmp, out)
    if module is not None:
        os.replace(ARGS_MODULE + ".tmp", ARGS_MODULE)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
