"""Build libvidkv.so (gfx950, hipcc) and, where there are a g++ and the headers of Python and torch, the binding's
native call layer (host) in-tree.  `python -m paper_2503_16257_amd.build`."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libvidkv.so")
MARSHAL = os.path.join(HERE, "vidkv_marshal.so")

SOURCES = ["vidkv_api.hip", "quant_keys.hip", "quant_keys_mfma.hip", "quant_values.hip",
           "quant_values_enc.hip", "decode_attn.hip", "decode_attn_mfma.hip", "decode_attn_mfma_b.hip",
           "decode_attn_mfma_c.hip", "decode_attn_mfma_t.hip", "saliency.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA results go to ordinary VGPRs (no accumulator-register moves)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-function",
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def _build_marshal() -> None:
    """csrc/marshal.cpp: a CPython extension that reads torch tensors (host code, no device code)."""
    import torch
    from .binding import native_tag
    t = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-I{sysconfig.get_paths()['include']}",
           "-isystem", f"{t}/include", "-isystem", f"{t}/include/torch/csrc/api/include",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DVIDKV_BUILT_FOR="{native_tag()}"',
           os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
           f"-L{t}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{t}/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on marshal.cpp:\n{r.stderr}")


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, SOURCES))
    built = [LIB]
    try:
        marshal.result()
        built.append(MARSHAL)
    except (ImportError, OSError, RuntimeError) as e:          # the binding works without it
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)                                 # (nor is one of an older source left)
        print(f"vidkv_marshal.so was not built, calls are marshalled in Python: {e}", file=sys.stderr)
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    if verbose:
        print(f"built {' and '.join(built)}")
    return LIB


if __name__ == "__main__":
    build()
