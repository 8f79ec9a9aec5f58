"""The fp32 kernels at the edges of their tiles: attention over key counts
around its 32-key tiles and four-way key split, with large logits and
NaN-filled V^T padding."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import assert_elementwise, attention_bound, need_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [2, 31, 32, 33, 64, 65, 96, 97, 128, 129, 161, 1013])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("std", [1.0, 6.0])
def test_attention_f32_tiles_and_key_split(L, d, std):
    P = need_gpu()
    nh = 3
    rng = np.random.default_rng(L * 7 + d)
    q, k = (rng.normal(size=(nh, L, d)).astype(np.float32) * std for _ in range(2))
    v = rng.normal(size=(nh, L, d)).astype(np.float32)
    ld = (L + 7) // 8 * 8 + 8
    vt = np.full((nh, d, ld), np.nan, np.float32)
    vt[:, :, :L] = v.transpose(0, 2, 1)
    o = torch.empty((L, nh * d), device="cuda")
    P.attention(to_dev(q), to_dev(k), to_dev(vt), o)
    again = torch.empty_like(o)
    P.attention(to_dev(q), to_dev(k), to_dev(vt), again)
    assert torch.equal(o, again)
    for j in range(nh):
        ref = O.attention(q[j], k[j], v[j])
        # a score's fp32 rounding (d products of size std^2 each) shifts its
        # probability by that much; attention_bound's share covers std = 1
        slack = 1.0 + 0.05 * std * std
        assert_elementwise(to_np(o[:, j * d:(j + 1) * d]), ref,
                           slack * attention_bound(q[j], k[j], v[j], False), 3e-5,
                           f"fp32 L={L} d={d} std={std} head {j}")


@pytest.mark.parametrize("d", [64, 128])
def test_attention_f32_masked_keys_have_no_weight(d):
    """A run of keys whose scores are all -inf (an additive mask carried in
    one channel) leaves the other keys' softmax: no NaN from a wave or a tile
    that sees only masked keys."""
    P = need_gpu()
    L, nh = 300, 1
    rng = np.random.default_rng(d)
    q, k, v = (rng.normal(size=(nh, L, d)).astype(np.float32) for _ in range(3))
    q[:, :, 0] = 1.0
    masked = np.zeros(L, bool)
    masked[64:200] = True           # whole 32-key tiles, on every wave
    k[:, masked, 0] = -np.inf
    vt = np.zeros((nh, d, 304), np.float32)
    vt[:, :, :L] = v.transpose(0, 2, 1)
    o = torch.empty((L, d), device="cuda")
    P.attention(to_dev(q), to_dev(k), to_dev(vt), o)
    ref = O.attention(q[0], k[0][~masked], v[0][~masked])
    np.testing.assert_allclose(to_np(o), ref, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 3, 17, 18, 19])
def test_attention_f32_few_keys(L, d, prescaled):
    """One wave per query up to 18 keys, the matrix kernel from 19 on; V^T's
    padding is NaN, more queries than a workgroup's four, a masked key."""
    P = need_gpu()
    nh = 5
    rng = np.random.default_rng(L + d)
    q, k, v = (rng.normal(size=(nh, L, d)).astype(np.float32) for _ in range(3))
    keep = np.ones(L, bool)
    if L > 3:
        q[:, :, 0] = 1.0
        k[:, 2, 0] = -np.inf
        keep[2] = False
    q_dev = (q * np.float32(P.q_scale(d))).astype(np.float32) if prescaled else q
    vt = np.full((nh, d, 24), np.nan, np.float32)
    vt[:, :, :L] = v.transpose(0, 2, 1)
    o = torch.empty((L, nh * d), device="cuda")
    P.attention(to_dev(q_dev), to_dev(k), to_dev(vt), o, q_prescaled=prescaled)
    for j in range(nh):
        kj, vj = k[j][keep], v[j][keep]
        assert_elementwise(to_np(o[:, j * d:(j + 1) * d]), O.attention(q[j], kj, vj),
                           1.05 * attention_bound(q[j], kj, vj, False), 3e-5,
                           f"fp32 few keys L={L} d={d} head {j}")


def test_attention_f32_more_heads_than_a_grid_dimension_holds():
    """One query of 2^24 + 3 heads: the few-keys kernel's workgroups fold into two
    grid dimensions."""
    P = need_gpu()
    nh, d = (1 << 24) + 3, 64
    q, k = (torch.ones((nh, 1, d), device="cuda") for _ in range(2))
    vt = torch.zeros((nh, d, 8), device="cuda")
    v = torch.arange(nh, device="cuda", dtype=torch.float32)[:, None] + 1.0
    vt[:, :, 0] = v
    o = torch.empty((1, nh * d), device="cuda")
    P.attention(q, k, vt, o)
    del q, k, vt
    # a weight of 1 after one rounding each of p, l and their quotient
    assert float((o.view(nh, d) / v - 1.0).abs().max()) <= 2.0 ** -21
    del o, v
    torch.cuda.empty_cache()


F32_KINDS = ["bias", "gelu", "gate_residual", "euler", "qkv"]


def _linear(P, kind, a, wt, bias, gate, base):
    M, N = a.shape[0], wt.shape[0]
    if kind == "qkv":  # 4 heads of 64, Q pre-scaled; returned token-major
        nh, d = N // 192, 64
        q, k = (torch.empty((nh, M, d), device="cuda") for _ in range(2))
        vt = torch.zeros((nh, d, (M + 7) // 8 * 8), device="cuda")
        P.linear(a, wt, P.ACID_EPI_QKV, bias, q=q, k=k, vt=vt, n_heads=nh, head_dim=d,
                 q_prescale=True)
        return torch.cat([q.permute(1, 0, 2).reshape(M, -1), k.permute(1, 0, 2).reshape(M, -1),
                          vt[:, :, :M].permute(2, 0, 1).reshape(M, -1)], 1)
    if kind in ("gate_residual", "euler"):
        out = base[:M].clone()
        if kind == "euler":
            P.linear(a, wt, P.ACID_EPI_EULER, bias, out=out, dsigma=-0.25)
        else:
            P.linear(a, wt, P.ACID_EPI_GATE_RESIDUAL, bias, gate=gate, out=out)
        return out
    out = torch.empty((M, N), device="cuda")
    P.linear(a, wt, P.ACID_EPI_BIAS_GELU if kind == "gelu" else P.ACID_EPI_BIAS, bias, out=out)
    return out


@pytest.mark.parametrize("kind", F32_KINDS)
@pytest.mark.parametrize("K", [128, 640])
def test_linear_f32_tiles_same_bits(kind, K):
    """32 x 32 tiles (few rows) and 64 x 64 tiles (many) sum in the same
    order: a call's rows are bit for bit the prefix of a larger call's.  The
    larger call against fp64; operands at 4-byte alignment give the same."""
    P = need_gpu()
    N, full = 768, 2100
    rng = np.random.default_rng(K)
    a = to_dev(rng.normal(size=(full, K)))
    wt = to_dev(rng.normal(size=(N, K)) / np.sqrt(K))
    bias, gate = to_dev(rng.normal(size=N) * 0.1), to_dev(rng.normal(size=N))
    base = to_dev(rng.normal(size=(full, N)))
    whole = _linear(P, kind, a, wt, bias, gate, base)
    y = to_np(a) @ to_np(wt).T + to_np(bias)
    acc = K * 2.0 ** -24 * (np.abs(to_np(a)) @ np.abs(to_np(wt)).T + np.abs(to_np(bias)))
    b, g = to_np(base), to_np(gate)
    ref, tol = {"bias": (y, acc), "gelu": (O.gelu_tanh(y), 1.13 * acc + 1e-6),
                "gate_residual": (b + g * y, np.abs(g) * acc + 2.0 ** -22 * (np.abs(b) + np.abs(g * y))),
                "euler": (b - 0.25 * y, 0.25 * acc + 2.0 ** -22 * (np.abs(b) + np.abs(y))),
                "qkv": (y * np.where(np.arange(N) < 256, P.q_scale(64), 1.0), acc)}[kind]
    assert_elementwise(to_np(whole), ref, tol, 2.0 ** -22, f"fp32 {kind} K={K}")
    for m in (1, 31, 32, 33, 130, 700, 2049):
        assert torch.equal(_linear(P, kind, a[:m].contiguous(), wt, bias, gate, base), whole[:m]), m
    flat = torch.empty(full * K + 1, device="cuda")
    off = flat[1:].view(full, K)
    off.copy_(a)
    assert off.data_ptr() % 16 == 4
    assert torch.equal(_linear(P, kind, off, wt, bias, gate, base), whole)
    assert torch.equal(_linear(P, kind, off[:45], wt, bias, gate, base), whole[:45])
