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
