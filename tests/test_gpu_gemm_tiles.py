"""The bf16 GEMM's output tiles (256 x 256, 256 x 128, 128 x 128, 64 x 64,
chosen by how many rounds of the CUs a launch takes): a token's outputs do
not depend on how many other tokens the call holds, so a call whose rows are
a prefix of a larger call's gives the same bits, whichever tile each takes.
The largest call is checked against fp64 on sampled rows."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from gemm_form_util import device_cus, gemm_form
from gpu_util import assert_elementwise, need_gpu, to_np

pytestmark = pytest.mark.gpu

D = 64


def _run(P, kind, a, wt, bias, gate, base, rows):
    a = a[:rows].contiguous()
    M, N = rows, wt.shape[0]
    if kind == "qkv":
        nh = N // (3 * D)
        q, k = (torch.empty((nh, M, D), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        vt = torch.zeros((nh, D, (M + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")
        P.linear(a, wt, P.ACID_EPI_QKV, bias, q=q, k=k, vt=vt, n_heads=nh, head_dim=D,
                 q_prescale=True)
        # token-major [M][3 H], as the plain product
        return torch.cat([q.permute(1, 0, 2).reshape(M, -1), k.permute(1, 0, 2).reshape(M, -1),
                          vt[:, :, :M].permute(2, 0, 1).reshape(M, -1)], 1)
    if kind == "gelu":
        out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        P.linear(a, wt, P.ACID_EPI_BIAS_GELU, bias, out=out)
    elif kind == "gate_residual":
        out = base[:M].clone()
        P.linear(a, wt, P.ACID_EPI_GATE_RESIDUAL, bias, gate=gate, out=out)
    elif kind == "euler":
        out = base[:M].clone()
        P.linear(a, wt, P.ACID_EPI_EULER, bias, out=out, dsigma=-0.25)
    else:
        out = torch.empty((M, N), device="cuda")
        P.linear(a, wt, P.ACID_EPI_BIAS, bias, out=out)
    return out


@pytest.mark.parametrize("kind", ["bias", "gelu", "gate_residual", "euler", "qkv"])
@pytest.mark.parametrize("N,K,full,rows", [
    # 256 x 256 for the full call and the rows below for each smaller tile; K of
    # two and of six stages (fewer than, and more than, the staging rings hold)
    (1536, 128, 9000, {"64x64": (1, 63, 64, 65, 1031), "128x128": (1559,),
                       "256x128": (4671, 4864)}),
    (1536, 384, 9000, {"64x64": (33, 257), "128x128": (1559,), "256x128": (4671,)}),
    # a half-width last feature tile of the 256 x 256 kernel
    (2176, 128, 60000, {"64x64": (31,), "128x128": (1031,)}),
    (2176, 384, 4100, {"64x64": (31,), "128x128": (1031,), "256x128": (2500,)}),
    (1152, 384, 7690, {"64x64": (257,), "128x128": (1801,), "256x128": (3601,)})])
def test_prefix_rows_same_bits_whatever_the_tile(kind, N, K, full, rows):
    if kind == "qkv" and N % (3 * D):
        pytest.skip("no head count gives this N")
    P = need_gpu()
    assert gemm_form(full, N, K, False, device_cus(), kind)[0] == "256x256"
    for tile, ms in rows.items():
        assert [gemm_form(m, N, K, False, device_cus(), kind)[0] for m in ms] == [tile] * len(ms)
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K)
    a = torch.randn((full, K), generator=g, device="cuda").bfloat16()
    wt = (torch.randn((N, K), generator=g, device="cuda") / math.sqrt(K)).bfloat16()
    bias = torch.randn(N, generator=g, device="cuda") * 0.1
    gate = torch.randn(N, generator=g, device="cuda")
    base = torch.randn((full, N), generator=g, device="cuda")
    whole = _run(P, kind, a, wt, bias, gate, base, full)
    at = np.unique(np.concatenate([np.random.default_rng(K).choice(full, 40, replace=False),
                                   [0, full - 1]]))
    y = to_np(a[at]) @ to_np(wt).T + to_np(bias)
    # K fp32 additions of exact products, and the epilogue's own roundings
    acc = K * 2.0 ** -24 * (np.abs(to_np(a[at])) @ np.abs(to_np(wt)).T + np.abs(to_np(bias)))
    b = to_np(base[at])
    ref, tol = {"bias": (y, acc), "gelu": (O.gelu_tanh(y), 1.13 * acc + 1e-6),
                "gate_residual": (b + to_np(gate) * y, np.abs(to_np(gate)) * acc + 2.0 ** -22 * (np.abs(b) + np.abs(y * to_np(gate)))),
                "euler": (b - 0.25 * y, 0.25 * acc + 2.0 ** -22 * (np.abs(b) + np.abs(y))),
                "qkv": (y * np.where(np.arange(N) < N // 3, P.q_scale(D), 1.0), acc)}[kind]
    rtol = 1.01 * 2.0 ** -8 if kind in ("gelu", "qkv") else 2.0 ** -22
    assert_elementwise(to_np(whole[at]), ref, tol, rtol, f"{kind} {full} x {N} x {K}")
    for m in sum(rows.values(), ()):
        got = _run(P, kind, a, wt, bias, gate, base, m)
        assert torch.equal(got, whole[:m]), (kind, m)


def test_k_split_step_repeats_bits():
    """The K split of a mostly idle last round (840 tiles of 256 x 256 over
    256 CUs, K = 12288: the second FFN GEMM of a 17776-token block) adds its
    partial sums in a fixed order: repeated blocks are bit-identical."""
    import acid_inputs as ai
    P = need_gpu()
    cfg = ai.COG5B.replace(n_blocks=1, n_steps=1)
    assert gemm_form(cfg.n_tokens, cfg.hidden, cfg.ffn, True, device_cus(),
                     "gate_residual") == ("256x256", 3, 72)
    m = P.Model(cfg, max_steps=1)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    for tid, (_, shape) in enumerate(ai.manifest(cfg)):
        m.load_tensor(tid, torch.randn(shape, generator=g, device="cuda") * 0.02)
    h0 = torch.randn((cfg.n_tokens, cfg.hidden), generator=g, device="cuda")
    mod6 = torch.randn((6, cfg.hidden), generator=g, device="cuda") * 0.3
    outs = []
    for _ in range(3):
        h = h0.clone()
        m.block_forward(0, mod6, h)
        outs.append(h)
    assert bool(torch.isfinite(outs[0]).all())
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
