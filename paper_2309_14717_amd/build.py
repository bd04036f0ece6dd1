"""Compile the HIP sources into the in-tree C-ABI shared library for gfx950.

Run as ``python -m paper_2309_14717_amd.build``.  hipcc cross-compiles without a GPU.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

NATIVE = "_native.so"  # the binding's native form, a Python extension module beside the library

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqalora_hip.so")
SOURCES = ["api.hip", "quantize.hip", "gemm_dq.hip", "adapter.hip", "smallt.hip", "smallt4.hip", "smallt4_f16.hip",
           "midt.hip", "glue.hip", "optim.hip", "probe.hip", "compensate.hip", "gemm_dq_192.hip",
           "grads.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LLVM = os.environ.get("HIP_CLANG_PATH", "/opt/rocm/llvm/bin")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


# Kernels that must compile with zero scratch memory: those whose waits on outstanding memory
# operations are counted by hand (a register spill would add scratch traffic to the same
# counter), and the adapter-gradient kernels, whose staging arrays once ended up in scratch
# unnoticed (a local array the compiler does not promote to registers costs a round trip to
# memory per element).
NO_SCRATCH = {"gemm_dq.hip": "gemm_dq_kernel", "gemm_dq_192.hip": "gemm_dq_kernel", "midt.hip": "midt_kernel", "smallt.hip": "smallt_kernel", "smallt4.hip": "smallt4_kernel", "smallt4_f16.hip": "smallt4_kernel",
              "adapter.hip": ("front_kernel", "front_wide_kernel"), "grads.hip": ("z_kernel", "finish_kernel", "fused_kernel", "du_kernel", "db_kernel", "tail_kernel")}


def _as_tuple(v):
    return v if isinstance(v, tuple) else (v,)


def _check_no_scratch(src: str, remarks: str) -> None:
    """Parse -Rpass-analysis=kernel-resource-usage remarks; fail on any scratch use."""
    name, bad = None, []
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "ScratchSize [bytes/lane]:" in line and name and any(k in name for k in _as_tuple(NO_SCRATCH[src])):
            if int(line.split("ScratchSize [bytes/lane]:")[1].split()[0]) != 0:
                bad.append(name)
    if bad:
        raise RuntimeError(f"{src}: kernels that must not use scratch memory do: {bad}")


def _device_code(obj: str) -> str:
    """Assembly listing of the gfx950 code inside a compiled object."""
    bundle, code = obj + ".bundle", obj + ".gfx950"
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + bundle, obj, obj + ".tmp"])
    subprocess.check_call([os.path.join(LLVM, "clang-offload-bundler"), "--type=bc", "--unbundle",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + bundle, "--output=" + code])
    text = subprocess.check_output([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", code], text=True)
    for f in (bundle, code, obj + ".tmp"):
        os.remove(f)
    return text


_WIDE_STORE = re.compile(r"\bbuffer_store_(?:dwordx[34]|format_xyzw?)\s+v\[[^\]]*\],\s*[^,]+,\s*s\[[^\]]*\],\s*([a-z]\w*)")


def _check_wide_stores(src: str, listing: str) -> None:
    """Refuse buffer stores of more than 64 bits with a scalar offset register: behind these the compiler lets
    a vector instruction overwrite the data registers at once, and wrong values have been stored."""
    bad = [line.strip() for line in listing.splitlines() if _WIDE_STORE.search(line)]
    if bad:
        raise RuntimeError(f"{src}: {len(bad)} wide buffer stores with a scalar offset register, the first: {bad[0]}")


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    if src in NO_SCRATCH:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout)
            raise subprocess.CalledProcessError(res.returncode, cmd)
        _check_no_scratch(src, res.stdout)
    else:
        subprocess.check_call(cmd)
    _check_wide_stores(src, _device_code(obj))
    return obj


def build_native() -> str:
    """Compile csrc/binding.cpp (host code: CPython and PyTorch headers; no GPU code)."""
    import torch
    root = os.path.dirname(torch.__file__)
    out = os.path.join(HERE, NATIVE)
    tmp = out + ".tmp%d" % os.getpid()
    subprocess.check_call([
        os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
        "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(),
        "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
        "-I/opt/rocm/include", "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "binding.cpp"), "-o", tmp,
        "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
        "-Wl,-rpath," + os.path.join(root, "lib")])
    os.replace(tmp, out)
    return out


def build(verbose: bool = False, extra_flags=(), variant: str = "") -> str:
    """Build the library.  `variant` names a measurement build (say, with -DQALORA_ABLATE=n in
    `extra_flags`): it goes to libqalora_hip.<variant>.so with objects of its own, so the
    library the tests and the product load is never replaced by it."""
    global OBJ
    lib = LIB if not variant else LIB[:-3] + "." + variant + ".so"
    obj_dir = OBJ if not variant else OBJ + "_" + variant
    os.makedirs(obj_dir, exist_ok=True)
    saved, OBJ = OBJ, obj_dir
    try:
        with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
            native = None if variant else ex.submit(build_native)
            objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    finally:
        OBJ = saved
    tmp = lib + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, lib)
    if native:
        native.result()
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    # python -m paper_2309_14717_amd.build [--variant NAME] [compiler flags ...]
    args = sys.argv[1:]
    name = ""
    if len(args) >= 2 and args[0] == "--variant":
        name, args = args[1], args[2:]
    build(verbose=True, extra_flags=args, variant=name)
