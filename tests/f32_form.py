"""The choice of tiles for fp32 products (csrc/gemm_f32_form.h, plain arithmetic), compiled on its own for the CPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_12636_amd", "csrc", "gemm_f32_form.h")
SOURCE = """#include "%s"
extern "C" void f32_form(int64_t M, int64_t N, int64_t K, int wgrad, int reach16, int *out) {
  const tmk::F32Form f = tmk::f32_form(M, N, K, wgrad, reach16);
  out[0] = f.tile, out[1] = f.split, out[2] = f.patches;
}
extern "C" int f32_split(int64_t M, int64_t N, int64_t K, int wgrad, int reach16) { return tmk::f32_split(M, N, K, wgrad, reach16); }
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "form.cpp"), os.path.join(d, "form.so")
        with open(src, "w") as f:
            f.write(SOURCE % HEADER)
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", lib, src], check=True)
        return ctypes.CDLL(lib)


def form(M, N, K, wgrad, reach16=True):
    """(tile, split, patches) of C[M,N] over K."""
    out = (ctypes.c_int * 3)()
    _lib().f32_form(*(ctypes.c_int64(v) for v in (M, N, K)), int(wgrad), int(reach16), out)
    return tuple(out)


def forms(T, N, K):
    """The three products of a linear map, forward, input gradient and weight gradient, as "tile/split", with "p" in patches."""
    return " ".join("%d/%d%s" % (t, s, "p" if p else "")
                    for t, s, p in (form(T, N, K, False), form(T, K, N, False), form(N, K, T, True)))


def split(M, N, K, wgrad, reach16=True):
    """Whether C[M,N] over K goes to the kernel on bf16 terms; form() holds where not."""
    return bool(_lib().f32_split(*(ctypes.c_int64(v) for v in (M, N, K)), int(wgrad), int(reach16)))


def splits(T, N, K):
    """Of the three products of a linear map: forward, input gradient, weight gradient."""
    return split(T, N, K, False), split(T, K, N, False), split(N, K, T, True)
