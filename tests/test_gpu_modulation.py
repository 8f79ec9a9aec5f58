"""The modulation table's fp32 products: rows around the 32-row blocks, an
embedding width that is no multiple of the 8-wide K groups, both grid forms
(few and many columns), and a table at 4-byte alignment."""
import numpy as np
import pytest
import torch

import acid_inputs as ai
import oracle as O
from gpu_util import make_model, need_gpu, rel_err, to_np

pytestmark = pytest.mark.gpu


def _ref(om, sig, H):
    out = []
    for s in sig:
        mod = om.modulation(float(s))
        out.append(np.concatenate([np.stack(mod["blocks"]).reshape(-1, H), mod["head"]]))
    return np.stack(out)


@pytest.mark.parametrize("freq_dim", [2, 6, 250, 256])
@pytest.mark.parametrize("n_blocks,hidden", [(1, 128), (3, 384), (8, 768)])
def test_modulation_rows_and_ragged_embedding(freq_dim, n_blocks, hidden):
    P = need_gpu()
    cfg = ai.TINY.replace(n_blocks=n_blocks, hidden=hidden, n_heads=hidden // 64, ffn=128,
                          n_video=4, freq_dim=freq_dim)
    m, params = make_model(P, cfg, max_steps=70, std=0.1)
    om = O.DiTModel(cfg, params)
    sig = np.linspace(1.0, 0.01, 70).astype(np.float32)
    ref = _ref(om, sig, hidden)
    whole = m.timestep_modulation(sig)
    # 4 products of up to 768 fp32 terms each, through two SiLUs
    assert rel_err(to_np(whole), ref) < 2e-6
    for n in (1, 2, 31, 32, 33, 64, 65):
        assert torch.equal(m.timestep_modulation(sig[:n]), whole[:n]), n


def test_modulation_table_at_float_alignment():
    P = need_gpu()
    cfg = ai.TINY
    m, _ = make_model(P, cfg, max_steps=4)
    sig = ai.sigmas(4)[:3]
    want = m.timestep_modulation(sig)
    flat = torch.zeros(want.numel() + 1, device="cuda")
    import ctypes as C
    s = np.ascontiguousarray(sig)
    P.check(P.lib().acid_timestep_modulation(
        m.h, s.ctypes.data_as(C.POINTER(C.c_float)), 3, C.c_void_p(flat[1:].data_ptr()),
        C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    assert torch.equal(flat[1:].view_as(want), want) and float(flat[0]) == 0.0
