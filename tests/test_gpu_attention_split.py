"""bf16 attention's key split (short sequences: the waves of a workgroup take
ranges of the key tiles and merge in LDS) against the definition, at tile
counts around the number of ranges, ragged and not; and the unsplit kernel at
the same short lengths, which many heads select."""
import numpy as np
import pytest
import torch

import oracle as O
from gemm_form_util import attn_ranges, device_cus
from gpu_util import BF16_U, assert_elementwise, attention_bound, bf16_values, need_gpu, to_dev, to_np
from test_gpu_kernels import prescale_q

pytestmark = pytest.mark.gpu


def _case(P, nh, L, d, prescaled, std=1.0, check=(0,), grow=False):
    rng = np.random.default_rng(L * 3 + d + nh)
    q, k, v = (bf16_values(rng.normal(size=(nh, L, d)).astype(np.float32) * s) for s in (std, std, 1.0))
    if grow:  # the reference moves within each range, by different amounts
        k = bf16_values(k * (1.0 + 6.0 * np.arange(L) / L)[None, :, None].astype(np.float32))
    q_dev = q
    if prescaled:
        q_dev, q = prescale_q(P, q, d, torch.bfloat16)
    ld = (L + 7) // 8 * 8
    vt = np.full((nh, d, ld), np.nan, np.float32)
    vt[:, :, :L] = v.transpose(0, 2, 1)
    args = [to_dev(t, torch.bfloat16) for t in (q_dev, k, vt)]
    outs = [torch.full((L, nh * d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    for o in outs:
        P.attention(*args, o, q_prescaled=prescaled)
    assert torch.equal(outs[0], outs[1]) and bool(torch.isfinite(outs[0]).all())
    for j in check:
        ref = O.attention(q[j], k[j], v[j])
        assert_elementwise(to_np(outs[0][:, j * d:(j + 1) * d]), ref, attention_bound(q[j], k[j], v[j]),
                           1.05 * BF16_U, f"{nh} heads L={L} d={d} head {j}")


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d", [64, 128])
# 1 to 9 tiles of 64 keys, with and without a ragged one (split from 128 on);
# 1037: 17 tiles
@pytest.mark.parametrize("nh", [2, 20])  # d = 64: four ranges, or two (from 833 tokens on)
@pytest.mark.parametrize("L", [1, 33, 64, 65, 128, 129, 192, 255, 256, 257, 320, 383, 576, 1037, 1408])
def test_split_over_key_ranges(L, nh, d, prescaled):
    want = 1 if L < 128 else 2 if d == 128 or (nh == 20 and L >= 833) else 4
    assert attn_ranges(d, nh, L, device_cus()) == want
    _case(need_gpu(), nh, L, d, prescaled, check=(0, 1))


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d", [64, 128])
def test_split_with_growing_scores(d, prescaled):
    _case(need_gpu(), 2, 700, d, prescaled, std=2.0, check=(0, 1), grow=True)


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d,nh", [(64, 1024), (128, 600)])
@pytest.mark.parametrize("L", [64, 130, 320])
def test_unsplit_at_short_lengths(L, d, nh, prescaled):
    assert attn_ranges(d, nh, L, device_cus()) == 1
    _case(need_gpu(), nh, L, d, prescaled, check=(0, nh // 2, nh - 1))


@pytest.mark.parametrize("d", [64, 128])
def test_split_range_of_masked_keys(d):
    """Keys masked by a -inf score (an additive mask carried in one channel)
    over whole key ranges: their ranges get no weight and no NaN."""
    P = need_gpu()
    L = 512
    rng = np.random.default_rng(d)
    q, k, v = (bf16_values(rng.normal(size=(1, L, d)).astype(np.float32)) for _ in range(3))
    q[:, :, 0] = 1.0
    masked = np.zeros(L, bool)
    masked[: L // 2] = True
    k[:, masked, 0] = -np.inf
    o = torch.empty((L, d), dtype=torch.bfloat16, device="cuda")
    vt = np.ascontiguousarray(v.transpose(0, 2, 1))
    P.attention(*(to_dev(t, torch.bfloat16) for t in (q, k, vt)), o)
    ref = O.attention(q[0], k[0][~masked], v[0][~masked])
    np.testing.assert_allclose(to_np(o), ref, rtol=2e-2, atol=2e-2)


def _masked_case(P, nh, L, d, prescaled, masked, value, far, check=(0,)):
    """Keys masked by the score `value` in one channel, all other scores near
    0 or, with far, near `far`: the oracle over the unmasked keys alone."""
    rng = np.random.default_rng(L + d + int(np.flatnonzero(masked)[0]))
    q, k, v = (bf16_values(rng.normal(size=(nh, L, d)).astype(np.float32)) for _ in range(3))
    q[:, :, :2] = 1.0
    k[:, :, 0] = np.where(masked, np.float32(value), np.float32(0.0))
    k[:, :, 1] = far
    k = bf16_values(k)
    q_dev = q
    if prescaled:
        q_dev, q = prescale_q(P, q, d, torch.bfloat16)
    vt = np.full((nh, d, (L + 7) // 8 * 8), np.nan, np.float32)
    vt[:, :, :L] = v.transpose(0, 2, 1)
    o = torch.empty((L, nh * d), dtype=torch.bfloat16, device="cuda")
    P.attention(*(to_dev(t, torch.bfloat16) for t in (q_dev, k, vt)), o, q_prescaled=prescaled)
    # A score is d additions in fp32 of products of size |far|, each rounded by
    # half a unit there; a weight and the row sum follow it.
    u = 2.0 ** -24 * abs(far) if far else 0.0
    slack = 2 * d * u / np.sqrt(d)
    for j in check:
        qj, kj, vj = q[j], k[j][~masked], v[j][~masked]
        bound = attention_bound(qj, kj, vj) + slack * O.attention(qj, kj, np.abs(vj))
        assert_elementwise(to_np(o[:, j * d:(j + 1) * d]), O.attention(qj, kj, vj), bound,
                           1.05 * BF16_U, f"{nh} heads L={L} d={d} masked from "
                           f"{int(np.flatnonzero(masked)[0])} {value} far {far} head {j}")


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("value", [-np.inf, -1e30, -1e6])
@pytest.mark.parametrize("far", [0.0, -16384.0])
def test_masked_tile_is_no_reference(value, far, d, prescaled):
    """A masked tile of 64 keys, at the start of each key range and between
    (512 keys: ranges of two tiles at d = 64, of four at d = 128), a masked
    range, a masked ragged tile (processed first), and the unsplit kernel."""
    P = need_gpu()
    L = 512
    assert attn_ranges(d, 2, L, device_cus()) == 256 // d and attn_ranges(d, 300, 150, device_cus()) == 1
    for t in range(8):
        at = np.zeros(L, bool)
        at[64 * t:64 * t + 64] = True
        _masked_case(P, 2, L, d, prescaled, at, value, far)
    for a, b in ((0, 256), (256, 512), (384, 512), (0, 500)):
        at = np.zeros(L, bool)
        at[a:b] = True
        _masked_case(P, 2, L, d, prescaled, at, value, far)
    at = np.zeros(500, bool)
    at[448:] = True
    _masked_case(P, 2, 500, d, prescaled, at, value, far)
    for n, a in ((150, 128), (192, 0), (192, 64)):  # 300 heads: more workgroups than CUs, no split
        at = np.zeros(n, bool)
        at[a:a + 64] = True
        _masked_case(P, 300, n, d, prescaled, at, value, far, check=(0, 299))


@pytest.mark.parametrize("prescaled", [False, True], ids=["plain-q", "prescaled-q"])
@pytest.mark.parametrize("d", [64, 128])
def test_no_key_left_is_nan(d, prescaled):
    """Rows whose scores are all -inf have no softmax: NaN, as 0 / 0."""
    P = need_gpu()
    q = torch.ones((2, 130, d), device="cuda", dtype=torch.bfloat16)
    k = torch.full((2, 130, d), -float("inf"), device="cuda", dtype=torch.bfloat16)
    vt = torch.ones((2, d, 136), device="cuda", dtype=torch.bfloat16)
    o = torch.zeros((130, 2 * d), device="cuda", dtype=torch.bfloat16)
    P.attention(q, k, vt, o, q_prescaled=prescaled)
    assert bool(o.isnan().all())
