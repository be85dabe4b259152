"""Build libago.so (HIP, gfx950 only) and the binding's native part in-tree with hipcc and g++.

    python -m paper_2212_01005_amd.build [--force]

Each source under csrc/ is compiled to csrc/obj/<name>.o (in parallel) and linked into
paper_2212_01005_amd/libago.so.  Nothing is JIT-compiled at run time.
"""

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "obj")
LIB = os.path.join(HERE, "libago.so")
PYCALL = os.path.join(HERE, "_agocall.so")

SOURCES = [
    "ago_host.cpp",
    "ago_graph.cpp",
    "ago_lower.cpp",
    "ago_plan.cpp",
    "ago_api.hip",
    "ago_elementwise.hip",
    "ago_gemm.hip",
    "ago_gemm_dma.hip",
    "ago_gemm_dma_rows.hip",
    "ago_gemm_dma_packed.hip",
    "ago_gemm_dma_special.hip",
    "ago_conv.hip",
    "ago_fused_invres.hip",
    "ago_invres_reg.hip",
    "ago_invres_reg_b13.hip",
    "ago_invres_reg_b15.hip",
    "ago_invres_reg_b23.hip",
    "ago_invres_reg_b25.hip",
    "ago_invres_reg_f13.hip",
    "ago_invres_reg_f15.hip",
    "ago_invres_reg_f23.hip",
    "ago_invres_reg_f25.hip",
    "ago_fused_conv_chain.hip",
    "ago_fused_ffn.hip",
    "ago_fused_ffn_stream.hip",
    "ago_fused_ffn_packed.hip",
    "ago_fused_dw_dw.hip",
    "ago_fused_attn.hip",
    "ago_fused_qkv.hip",
]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    # keep hipcc from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _deps_mtime():
    hdrs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    hdrs.append(os.path.join(HERE, "..", "include", "ago.h"))
    return max(os.path.getmtime(h) for h in hdrs)


def _compile(src, force):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if (not force and os.path.exists(obj)
            and os.path.getmtime(obj) >= max(os.path.getmtime(path), _deps_mtime())):
        return obj, False
    cmd = [HIPCC] + FLAGS + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj, True


def _build_pycall(force):
    """The binding's native marshalling: host code against the Python and torch headers, linked to libago.so."""
    src = os.path.join(CSRC, "ago_pycall.cpp")
    if not force and os.path.exists(PYCALL) and os.path.getmtime(PYCALL) >= max(os.path.getmtime(src), _deps_mtime()):
        return
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    cmd += ["-isystem" + d for d in [sysconfig.get_paths()["include"], os.path.join(rocm, "include")] + include_paths()]
    cmd += [src, "-o", PYCALL, "-L" + tlib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python",
            "-L" + HERE, "-l:libago.so", "-Wl,-rpath,$ORIGIN"]
    subprocess.check_call(cmd)


def build(force: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(lambda s: _compile(s, force), SOURCES))
    objs = [o for o, _ in results]
    if force or any(c for _, c in results) or not os.path.exists(LIB):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
        subprocess.check_call(cmd)
    _build_pycall(force)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
