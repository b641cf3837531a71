"""Build libxred.so for gfx950 with hipcc (in-tree, no JIT cache).

    python -m paper_2510_20171_amd.build

Every .hip file under csrc/ is compiled to an object in parallel, then linked
into paper_2510_20171_amd/libxred.so; ceiling/xred_ceiling.hip (a measuring
tool for bench.py) becomes paper_2510_20171_amd/libxred_ceiling.so, and
csrc/xred_torch.cpp (host code, the host compiler) the Python module
_xred_torch.so the binding marshals tensors with.  That module is left out,
with a note, where g++, Python.h or torch's headers are missing: the library
needs none of them.  Flags of the HIP code:
  --offload-arch=gfx950      MI355X only
  -ffp-contract=off          no fused multiply-add: one IEEE op per float op
  -fno-gpu-flush-denormals-to-zero   binary32 subnormals are kept
  -packed-fp32-ops (off)     no v_pk_{add,mul,fma}_f32 generated
  -fvisibility=hidden        only the xred_* C ABI is exported
  -mllvm -amdgpu-atomic-optimizer-strategy=None
                             single-lane atomics stay single-lane: the
                             optimizer turns them into wave-wide sequences
                             that wait for the atomic's result at once
                             (the batched queue claims tiles ahead)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
OUT = PKG / "libxred.so"
# the traffic-only ceiling kernel bench.py measures beside libxred (its own
# library: not part of libxred's interface)
CEILING_SRC = PKG / "ceiling" / "xred_ceiling.hip"
CEILING_OUT = PKG / "libxred_ceiling.so"
# the binding's tensor marshalling (a CPython module against torch's headers)
TORCH_SRC = CSRC / "xred_torch.cpp"
TORCH_OUT = PKG / "_xred_torch.so"
BUILD = PKG / "_build"
HIPCC = "/opt/rocm/bin/hipcc"

HIPFLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-ffp-contract=off", "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wno-unused-function",
]


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the gfx950 feature name; that warning is noise
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "not a recognized feature for this target" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"command failed: {' '.join(cmd)}\n{err}")
    if err.strip():
        print(err, file=sys.stderr)


def _torch_module_cmd(out: Path):
    """The command that builds the marshalling module; ImportError names what is missing."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    gxx = shutil.which("g++")
    if gxx is None:
        raise ImportError("g++ is missing")
    incs = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]
    for header in ("Python.h", "torch/csrc/autograd/python_variable.h"):
        if not any((Path(i) / header).exists() for i in incs):
            raise ImportError(f"{header} is missing")
    lib = Path(torch.__file__).resolve().parent / "lib"
    return [gxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *(x for i in incs for x in ("-isystem", i)), str(TORCH_SRC), "-o", str(out),
            f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{lib}"]


def build(jobs: int = 0, verbose: bool = False) -> Path:
    """Compile every csrc/*.hip and link libxred.so; returns its path."""
    BUILD.mkdir(exist_ok=True)
    sources = sorted(CSRC.glob("*.hip"))
    objs = [BUILD / (s.stem + ".o") for s in sources]
    cmds = [[HIPCC, *HIPFLAGS, "-c", str(s), "-o", str(o)] for s, o in zip(sources, objs)]
    ceiling_tmp = CEILING_OUT.with_suffix(".so.tmp")
    cmds.append([HIPCC, *HIPFLAGS, "-shared", str(CEILING_SRC), "-o", str(ceiling_tmp)])
    torch_tmp = TORCH_OUT.with_suffix(".so.tmp")
    try:
        cmds.append(_torch_module_cmd(torch_tmp))
    except ImportError as e:
        print(f"{TORCH_OUT.name} is not built ({e}): calls will be marshalled in Python",
              file=sys.stderr)
        TORCH_OUT.unlink(missing_ok=True)
        torch_tmp = None
    if jobs <= 0:
        jobs = min(16, os.cpu_count() or 4)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(_run, cmds))
    tmp = OUT.with_suffix(".so.tmp")
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *map(str, objs), "-o", str(tmp)])
    tmp.replace(OUT)
    ceiling_tmp.replace(CEILING_OUT)
    if torch_tmp is not None:
        torch_tmp.replace(TORCH_OUT)
    if verbose:
        print(f"built {OUT}{f', {TORCH_OUT}' if torch_tmp else ''} and {CEILING_OUT}")
    return OUT


if __name__ == "__main__":
    build(verbose=True)
