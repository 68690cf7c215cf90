"""Builds libspecvlm.so (hand-written HIP for gfx950) in-tree with hipcc, and the binding's native part
(_specvlm_native.so, host code only) with g++."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libspecvlm.so")
NATIVE = os.path.join(HERE, "_specvlm_native.so")
SOURCES = ["api.hip", "sample_kernels.hip", "accept_sample.hip", "draft_tree.hip", "head_argmax.hip", "compress.hip", "attn_valu.hip", "attn_mfma.hip", "attn_wave.hip", "attn_streams.hip"]


HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + INCLUDE, "-I" + CSRC,
               # compiler-generated packed fp32 ops are switched off on the test machines
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               # keep MFMA accumulators in architectural VGPRs: the attention kernel rescales and
               # converts them with VALU ops, and AGPR copies would dominate its inner loop
               "-mllvm", "-amdgpu-mfma-vgpr-form"]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def native_command() -> list[str]:
    """The binding's native part: a CPython extension over torch's C++ tensors."""
    import torch
    t = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(t, "include"), os.path.join(t, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I" + INCLUDE, "-I" + sysconfig.get_paths()["include"],
            "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
            os.path.join(CSRC, "native_binding.cpp"), "-o", NATIVE,
            "-L" + lib, "-Wl,-rpath," + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def _run(cmd: list[str]) -> str:
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + proc.stdout + proc.stderr)
    return proc.stderr


def build(verbose: bool = False) -> str:
    """Compile every kernel for gfx950 (cross-compiles without a GPU), one process per source file.
    Always rebuilds."""
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=8) as pool:
            native = pool.submit(_run, native_command())
            said = list(pool.map(_run, [[_hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, s), "-o", o]
                                        for s, o in zip(SOURCES, objs)]))
            said.append(_run([_hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB, *objs]))
            said.append(native.result())
    if verbose:
        print("".join(said))
    return LIB


def kernel_resource_usage(source: str) -> dict:
    """Per-kernel VGPR count, scratch bytes per lane and LDS bytes of one source file, from the
    compiler's own kernel-resource-usage remarks (device code only, nothing is linked)."""
    import re
    with tempfile.TemporaryDirectory() as tmp:
        said = _run([_hipcc(), *HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
                     "-o", os.path.join(tmp, "k.o"), os.path.join(CSRC, source)])
    out, name = {}, None
    for line in said.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            out[name] = {}
        for key, pat in (("vgprs", r"\bVGPRs: (\d+)"), ("scratch", r"ScratchSize \[bytes/lane\]: (\d+)"),
                         ("lds", r"LDS Size \[bytes/block\]: (\d+)")):
            m = re.search(pat, line)
            if m and name:
                out[name][key] = int(m.group(1))
    return out


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(INCLUDE, "specvlm.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build(verbose=True))
