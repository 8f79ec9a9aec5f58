"""The K split of the smaller bf16 GEMM tiles (few rows and a long K, inside a
model, which holds the partial sums): one block against plain fp64 on the same
weights, and the same bits when it runs again."""
import math

import pytest
import torch

import acid_inputs as ai
from gemm_form_util import device_cus, gemm_form
from gpu_util import BF16_U, assert_close_to_scale, need_gpu, rel_err, to_np

pytestmark = pytest.mark.gpu


def _ln(x, shift, scale):
    x = x - x.mean(-1, keepdim=True)
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * (1 + scale) + shift


def _block(h, w, mod, heads, d, parallel):
    """One block in fp64; w: (qkv, o, f1, f2) weights [in][out] and biases."""
    (wq, bq), (wo, bo), (w1, b1), (w2, b2) = w
    a = _ln(h, mod[0], mod[1])
    q, k, v = (a @ wq + bq).split(heads * d, 1)
    o = torch.empty_like(h)
    for j in range(heads):
        i = slice(j * d, (j + 1) * d)
        o[:, i] = torch.softmax(q[:, i] @ k[:, i].t().contiguous() / math.sqrt(d), -1) @ v[:, i]
    o = o @ wo + bo

    def mlp(z):
        return torch.nn.functional.gelu(z @ w1 + b1, approximate="tanh") @ w2 + b2

    if parallel:
        return h + mod[2] * (o + mlp(a))
    h = h + mod[2] * o
    return h + mod[5] * mlp(_ln(h, mod[3], mod[4]))


# rows and widths, and the tile and K split of the block's products (Q K V,
# output, FFN1, FFN2; parallel: Q K V and FFN1, output and FFN2): 64 x 64 tiles in
# 8 and 3 ranges (one row, a ragged row tile), 128 x 128 and 256 x 128 tiles (full
# and ragged), ranges of unequal length (70 and 140 K-steps in 8, 3, 7 and 5),
# the output projection and the GELU product at hidden 4096, the fused Q K V and
# GELU product, and 256 x 256 tiles whose last round is split (Q K V, output).
@pytest.mark.parametrize("rows,heads,d,ffn,form,tiles", [
    (1, 4, 64, 8192, "sequential", "64x64/1 64x64/1 64x64/1 64x64/8"),
    (65, 8, 64, 4480, "sequential", "64x64/1 64x64/1 64x64/1 64x64/8"),
    (130, 12, 128, 8960, "sequential", "64x64/1 64x64/1 64x64/1 64x64/3"),
    (300, 12, 128, 8960, "sequential", "64x64/1 64x64/1 128x128/1 128x128/7"),
    (1000, 12, 128, 8960, "sequential", "64x64/1 64x64/1 256x256/1 256x128/5"),
    (1280, 12, 128, 8960, "parallel", "256x128/1 256x128/4"),
    (100, 32, 128, 512, "sequential", "128x128/2 64x64/2 64x64/8 64x64/1"),
    (64, 32, 128, 256, "sequential", "64x64/1 64x64/4 64x64/8 64x64/1"),
    (100, 30, 128, 4096, "parallel", "128x128/2 128x128/8"),
    (1500, 32, 128, 256, "sequential", "256x256/2 256x128/1 64x64/2 256x128/1"),
    (4680, 32, 128, 256, "sequential", "256x256/1 256x256/2 128x128/3 256x256/1"),
])
def test_block_with_split_products(rows, heads, d, ffn, form, tiles):
    P = need_gpu()
    H = heads * d
    prods = [("qkv", 3 * H, H), ("gate_residual", H, H), ("gelu", ffn, H),
             ("gate_residual", H, ffn)] if form == "sequential" else \
        [("qkv_gelu", 3 * H + ffn, H), ("gate_residual", H, H + ffn)]
    assert " ".join("%s/%d" % gemm_form(rows, n, k, True, device_cus(), kind)[:2]
                    for kind, n, k in prods) == tiles
    cfg = ai.TINY.replace(dtype="bf16", n_blocks=1, hidden=H, n_heads=heads, head_dim=d, ffn=ffn,
                          n_video=rows, n_text=0, block=form)
    m = P.Model(cfg, max_steps=1)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + H)
    keep = {}
    for k, (name, shape) in enumerate(ai.manifest(cfg)):
        t = torch.randn(shape, generator=g, device="cuda") * 0.02
        m.load_tensor(k, t)
        if 6 <= k < 14:
            keep[k] = (t.bfloat16() if len(shape) == 2 else t).double()
    h0 = torch.randn((rows, H), generator=g, device="cuda")
    mod = torch.randn((6, H), generator=g, device="cuda") * 0.3
    h, again = h0.clone(), h0.clone()
    m.block_forward(0, mod, h)
    m.block_forward(0, mod, again)
    assert torch.equal(h, again)
    w = [(keep[k], keep[k + 1]) for k in (6, 8, 10, 12)]
    ref = _block(h0.double(), w, mod.double(), heads, d, form == "parallel")
    assert_close_to_scale(to_np(h), ref.cpu().numpy(), True, f"{rows} rows H {H} F {ffn} {form}")
    # The update alone, whose scale is the products' own, in 2-norm: at most
    # four roundings to bf16 in series on a branch (LN, QKV, probabilities,
    # attention output), each at most 2^-8 of its value.
    assert rel_err(to_np(h - h0), (ref - h0.double()).cpu().numpy()) <= 4 * BF16_U
