"""Build libepp.so (HIP, gfx950) and the CPython extension of its per-pass calls, in-tree."""
from __future__ import annotations

import hashlib
import shutil
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
SO = PKG / "libepp.so"
BINDING = PKG / ("_binding" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = sorted((PKG / "csrc").glob("*.hip"))
BINDING_SOURCE = PKG / "csrc" / "epp_binding.cpp"

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


STAMP = PKG / "libepp.so.sources"  # hash of the sources the library file was built from


def source_hash() -> str:
    """Hash of everything under csrc/ (names and contents)."""
    h = hashlib.sha256()
    for f in sorted((PKG / "csrc").glob("*")):
        h.update(f.name.encode())
        h.update(f.read_bytes())
    return h.hexdigest()[:16]


def _run(cmd: list, verbose: bool) -> None:
    if verbose:
        print(" ".join(map(str, cmd)), flush=True)
    subprocess.check_call([str(c) for c in cmd])


def hip_object(src: Path, obj: Path, verbose: bool = False) -> None:
    _run(["hipcc", *HIPCC_FLAGS, f"-I{ROOT / 'include'}", f"-I{PKG / 'csrc'}", "-c", src, "-o", obj], verbose)


def link_library(objects: list, verbose: bool = False) -> None:
    _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", SO], verbose)


def binding_object(obj: Path, verbose: bool = False) -> None:
    import torch
    inc = Path(torch.__file__).parent / "include"
    rocm = Path(shutil.which("hipcc") or "/opt/rocm/bin/hipcc").resolve().parent.parent
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", f"-I{ROOT / 'include'}", f"-isystem{inc}",
          f"-isystem{rocm / 'include'}",
          f"-isystem{inc / 'torch/csrc/api/include'}", f"-I{sysconfig.get_paths()['include']}", "-c", BINDING_SOURCE,
          "-o", obj], verbose)


def link_binding(obj: Path, verbose: bool = False) -> None:
    """Linked with libepp.so beside it and with the libraries of the PyTorch that runs it."""
    import torch
    lib = Path(torch.__file__).parent / "lib"
    _run(["g++", "-shared", "-fPIC", obj, f"-L{PKG}", "-l:libepp.so", f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
          "-Wl,--allow-shlib-undefined", "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{lib}", "-o", BINDING], verbose)


def build(verbose: bool = False) -> Path:
    stamp = source_hash()
    for old in (STAMP, SO, BINDING):  # (a process that has them loaded keeps its own)
        old.unlink(missing_ok=True)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(4) as pool:
        objects = [Path(tmp) / (s.stem + ".o") for s in SOURCES]
        binding = Path(tmp) / "binding.o"
        jobs = [pool.submit(hip_object, s, o, verbose) for s, o in zip(SOURCES, objects)]
        jobs.append(pool.submit(binding_object, binding, verbose))
        for j in jobs:
            j.result()
        link_library(objects, verbose)
        link_binding(binding, verbose)
    STAMP.write_text(stamp + "\n")  # (a library left over from other sources is then recognisable)
    return SO


if __name__ == "__main__":
    build(verbose=True)
