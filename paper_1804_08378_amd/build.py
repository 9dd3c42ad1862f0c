"""Build libbrainslug_hip.so (hipcc, gfx950) in-tree, next to this file."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbrainslug_hip.so")
TORCH_EXT = os.path.join(HERE, "_bs_torch.so")  # the binding's native calls (csrc/bs_torch.cpp, host code only)
SOURCES = ["bs_stack.cpp", "bs_plan.cpp", "bs_run.cpp", "bs_jit.cpp", "bs_trace.cpp", "bs_kernels.hip", "bs_lds.hip", "bs_rows.hip",
           "bs_rows2.hip", "bs_xrows.hip", "bs_chain.hip", "bs_chain_window.hip", "bs_chain_nhwc.hip", "bs_chain_window_nhwc.hip", "bs_nhwc.hip", "bs_nhwc_tile.hip", "bs_nhwc_rows.hip", "bs_strip.hip", "bs_pool_band.hip", "bs_backward.cpp", "bs_backward.hip", "bs_backward_strip.hip", "bs_probe.hip"]
# device headers whose text is embedded in the library for run-time (hipRTC) kernel builds
JIT_HEADERS = ["bs_kargs.h", "bs_device.h", "bs_lds_device.h", "bs_rows_device.h", "bs_xrows_device.h", "bs_chain_device.h", "bs_chain_window_device.h"]

# -ffp-contract=off: the only fused multiply-add is the explicit one of BatchNorm.
# packed-fp32 instructions are disabled for the device code.
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-ffp-contract=off",
         "-fno-fast-math", "-fvisibility=hidden", "-Wall", "-Wextra", "-Wno-unused-parameter",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the by-value kernel argument blocks are read in place (kernarg segment) only if the
         # optimizer may look through all their uses; the default cap is too low for the LDS kernel
         "-mllvm", "-instcombine-max-copied-from-constant-users=100000",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def torch_tag() -> str:
    """What the native calls are compiled for (the text stands in the built file); "" where torch is not installed."""
    import importlib.metadata
    import sysconfig
    try:
        version = importlib.metadata.version("torch")
    except importlib.metadata.PackageNotFoundError:
        try:  # a torch that was not installed as a package
            from torch import __version__ as version
        except ImportError:
            return ""
    return "bs_torch for torch %s, %s;" % (version, sysconfig.get_config_var("SOABI"))


def torch_ext_fits() -> bool:
    """Are the native calls there, and built for the installed torch and this Python?"""
    tag = torch_tag()
    if not tag or not os.path.exists(TORCH_EXT):
        return False
    with open(TORCH_EXT, "rb") as f:
        return tag.encode() in f.read()


def up_to_date() -> bool:
    if not os.path.exists(LIB):
        return False
    if torch_tag() and (not torch_ext_fits() or os.path.getmtime(TORCH_EXT) < os.path.getmtime(os.path.join(CSRC, "bs_torch.cpp"))):
        return False
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, h) for h in JIT_HEADERS + ["bs_internal.h", "bs_rows_tables.h", "bs_nhwc_device.h", "bs_bwd_device.h", "bs_strip_device.h", "bs_backward_keys.h"]]
    deps.append(os.path.join(ROOT, "include", "brainslug.h"))
    return all(os.path.getmtime(d) <= t for d in deps)


def write_embedded_headers(path: str) -> None:
    """C++ source holding the text of the device headers (what run-time builds compile from)."""
    parts = ["// generated by build.py from csrc/*.h: do not edit\n", "namespace bs {\n",
             "struct EmbeddedHeader {\n    const char *name, *text;\n};\n",
             "extern const EmbeddedHeader k_jit_headers[];\nextern const int k_jit_n_headers;\n",
             "const EmbeddedHeader k_jit_headers[] = {\n"]
    for h in JIT_HEADERS:
        text = open(os.path.join(CSRC, h)).read()
        assert ')BSJIT"' not in text
        # string literals are limited in length by some compilers: split into chunks
        chunks = [text[i:i + 8000] for i in range(0, len(text), 8000)]
        lit = "\n".join('R"BSJIT(%s)BSJIT"' % c for c in chunks)
        parts.append('    {"%s",\n%s},\n' % (h, lit))
    parts.append("};\nconst int k_jit_n_headers = %d;\n}  // namespace bs\n" % len(JIT_HEADERS))
    new = "".join(parts)
    if not os.path.exists(path) or open(path).read() != new:
        with open(path, "w") as f:
            f.write(new)


def build_torch_ext() -> None:
    """Compile csrc/bs_torch.cpp against the installed torch (its headers and libraries; nothing of it runs on the device)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = TORCH_EXT + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wno-unused-parameter",
           "-DBS_TORCH_TAG=\"%s\"" % torch_tag(), "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for d in [*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "bs_torch.cpp"), "-o", tmp, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    subprocess.run(cmd, check=True)
    os.replace(tmp, TORCH_EXT)


def try_torch_ext() -> bool:
    """The native calls are optional: the library needs no torch, and the binding's Python code takes every call without them.  A file that
    cannot be built anew is removed, so that none for another torch or an older source stays."""
    try:
        build_torch_ext()
        return True
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(TORCH_EXT):
            os.remove(TORCH_EXT)
        print("without the native calls (%s): torch calls go through ctypes: %s" % (os.path.basename(TORCH_EXT), e), file=sys.stderr)
        return False


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and up_to_date():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    # BS_EXTRA_HIPCC_FLAGS: extra compiler flags (e.g. -D overrides of the tuning constants in bs_kargs.h)
    compile_flags = [f for f in FLAGS if f != "-shared"] + os.environ.get("BS_EXTRA_HIPCC_FLAGS", "").split()

    def compile_one(src):
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        cmd = [hipcc, *compile_flags, "-x", "hip", "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True)
        return obj

    embed = os.path.join(objdir, "bs_jit_embed.cpp")
    write_embedded_headers(embed)

    from concurrent.futures import ThreadPoolExecutor
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        ext = ex.submit(try_torch_ext)
        objs = list(ex.map(compile_one, sources() + [embed]))
        ext.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fvisibility=hidden", *objs, "-lhiprtc", "-ldl",
                    "-o", tmp], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
