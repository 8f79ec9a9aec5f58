"""The output tile and K split that a bf16 GEMM launch takes, from the
library's own rule (csrc/gemm_form.h compiled for the host), so that a test
can state which kernel its sizes reach."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES = ("256x256", "256x128", "128x128", "64x64")

SRC = """
#include "gemm_form.h"
extern "C" void form(int64_t M, int N, int K, int ws, int64_t cus, int64_t* out) {
  const acid::Form f = acid::choose_form(M, N, K, ws != 0, cus);
  out[0] = (int)f.tile;
  out[1] = f.split;
  out[2] = f.rem;
}
"""


@functools.lru_cache(None)
def _lib():
    d = tempfile.mkdtemp()
    src, so = os.path.join(d, "form.cpp"), os.path.join(d, "form.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2607_12358_amd", "csrc"), src, "-o", so], check=True)
    return C.CDLL(so)


def gemm_form(M, N, K, workspace=False, cus=256):
    """(tile, K split, tail tiles that the split applies to; 0: all)"""
    out = (C.c_int64 * 3)()
    _lib().form(C.c_int64(M), N, K, int(workspace), C.c_int64(cus), out)
    return TILES[out[0]], int(out[1]), int(out[2])


def device_cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count
