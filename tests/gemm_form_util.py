"""The output tile and K split that a bf16 GEMM launch takes, and the key
ranges of a bf16 attention launch, from the library's own rules
(csrc/gemm_form.h, csrc/attn_form.h compiled for the host), so that a test can
state which kernel its sizes reach."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES = ("256x256", "256x128", "128x128", "64x64")

SRC = """
#include "attn_form.h"
#include "gemm_form.h"
extern "C" int ranges(int d, int64_t n_heads, int64_t L, int64_t cus) {
  return acid::attn_key_ranges(d, n_heads, L, cus);
}
extern "C" void form(int epi, int64_t M, int N, int K, int ws, int64_t cus, int64_t* out) {
  const acid::Form f = acid::choose_form((acid::Out)epi, M, N, K, ws != 0, cus);
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


EPILOGUES = {"bias": 0, "gelu": 1, "gate_residual": 2, "euler": 2, "qkv": 3, "qkv_prescaled": 3,
             "qkv_gelu": 3}


def gemm_form(M, N, K, workspace=False, cus=256, kind="bias"):
    """(tile, K split, tail tiles that the split applies to; 0: all)"""
    out = (C.c_int64 * 3)()
    _lib().form(EPILOGUES[kind], C.c_int64(M), N, K, int(workspace), C.c_int64(cus), out)
    return TILES[out[0]], int(out[1]), int(out[2])


def attn_ranges(d, n_heads, L, cus=256):
    """Key ranges that the waves of a workgroup take (1: not split)"""
    return _lib().ranges(d, C.c_int64(n_heads), C.c_int64(L), C.c_int64(cus))


def device_cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count
