"""Builds libqfc.so (HIP, gfx950 only) in-tree with hipcc.

Usage: python -m paper_2505_00232_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqfc.so")
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))  # (another Python does not take it for its own)
MARSHAL_FOR = os.path.join(OBJ, "marshal_built_for")
SOURCES = ["api.hip", "pack.hip", "gemv.hip", "gemv_q8.hip", "actquant.hip", "rmsnorm.hip", "attention.hip", "gemm_i8.hip", "gemm_f16.hip", "gemm_skinny.hip", "probe.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed-fp32 code generation is switched off on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# Prefill attention holds the sums of the second product in accumulation registers, but its scores are vector operands at once:
# with every MFMA writing accumulation registers they would be moved over one by one (us with / without: head size 256, 2048 tokens
# 50.6 / 62.0; 128 and 64 level, and so is the kernel for few query rows in the same file, within the 1 % of two runs).
SOURCE_FLAGS = {"attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


# Kernels that load MFMA operands into registers with hand-written asynchronous loads and place the
# waits themselves: the compiler takes a destination register to be valid right after the load
# instruction, so if it spilled one it would save the stale value.  The build refuses any spill
# in these kernels (mangled-name fragments per source file).
NO_SPILL = {"gemm_i8.hip": ("gemm_i8_dw_kernel",)}


def _spilling_kernels(remarks: list[str], fragments: tuple[str, ...]) -> list[str]:
    """Names of the kernels matching `fragments` whose resource-usage remarks report scratch memory."""
    import re
    bad, name = [], None
    for line in remarks:
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            continue
        m = re.search(r"(ScratchSize \[bytes/lane\]|VGPRs Spill|SGPRs Spill): (\d+)", line)
        if m and name and any(f in name for f in fragments) and int(m.group(2)) != 0 and name not in bad:
            bad.append(name)
    return bad


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _deps() -> list[str]:
    """What the library is built from: the sources, the public headers, and this file with its flags."""
    include = os.path.join(HERE, "..", "include")
    return [os.path.join(d, f) for d in (CSRC, include) for f in os.listdir(d)] + [os.path.abspath(__file__)]


def _deps_newer(target: str) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in _deps())


def _marshal_stale() -> bool:
    """Older than what it is built from, or built against another Python or torch."""
    from .binding import _built_for
    if _deps_newer(MARSHAL) or not os.path.exists(MARSHAL_FOR):
        return True
    with open(MARSHAL_FOR) as f:
        return f.read() != _built_for()


def _build_marshal() -> None:
    """The host module behind the binding's most frequent calls, against torch's own headers (no device code).  The library and the binding do without it
    where it cannot be built."""
    import torch

    from .binding import _built_for
    root = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DQFC_BUILT_FOR="{_built_for()}"',
           *(f"-I{d}" for d in (f"{root}/include", f"{root}/include/torch/csrc/api/include", sysconfig.get_paths()["include"])),
           os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, f"-L{root}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{root}/lib"]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed = r.stderr if r.returncode != 0 else ""
    except OSError as e:
        failed = str(e)
    if failed:
        warnings.warn("marshal.cpp could not be built, calls cost about 1 us more:\n" + failed, RuntimeWarning, stacklevel=2)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)
    with open(MARSHAL_FOR, "w") as f:
        f.write(_built_for())


def build(force: bool = False, verbose: bool = False) -> str:
    library, marshal = force or _deps_newer(LIB), force or _marshal_stale()
    if not library and not marshal:
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    cc = _hipcc() if library else None

    def compile_one(src: str) -> str:
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        cmd = [cc, *FLAGS, *SOURCE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        if src in NO_SPILL:
            cmd.append("-Rpass-analysis=kernel-resource-usage")
        r = subprocess.run(cmd, capture_output=True, text=True)
        lines = r.stderr.splitlines()
        if src in NO_SPILL:
            spilled = _spilling_kernels(lines, NO_SPILL[src])
            lines = [l for l in lines if "-Rpass-analysis=kernel-resource-usage" not in l]
            if r.returncode == 0 and spilled:
                raise RuntimeError(f"{src}: register spills in {', '.join(spilled)} (their loads complete behind the compiler's back)")
        err = "\n".join(l for l in lines if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err)
        return obj

    with ThreadPoolExecutor(max_workers=7) as ex:
        module = ex.submit(_build_marshal) if marshal else None
        objs = list(ex.map(compile_one, SOURCES if library else []))
        if module:
            module.result()
    if not library:
        return LIB
    r = subprocess.run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
