"""Signals returned to the host through the models' shared page of pinned
memory: models beyond its 64 slots (which copy from the device instead) give
the same values, slots of destroyed models are handed out again, and two
models used from two threads and streams do not see each other's results."""
import threading

import pytest
import torch

import acid_inputs as ai
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

CFG = ai.TINY.replace(n_steps=2)


def _model(P, seed=0):
    m = P.Model(CFG, max_steps=2)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    for tid, (_, shape) in enumerate(ai.manifest(CFG)):
        m.load_tensor(tid, torch.randn(shape, generator=g, device="cuda") * 0.02)
    return m


def test_more_models_than_slots_and_reuse():
    P = need_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x, p, c = (torch.randn((CFG.n_video, CFG.hidden), generator=g, device="cuda") for _ in range(3))
    m_cur = torch.empty_like(x)
    for _ in range(2):  # the second round takes the slots the first gave back
        models = [_model(P) for _ in range(70)]
        sums = {m.l1_norms(x, p, c) for m in models}
        drifts = {m.drift_signal(x, 0.7, p, m_cur) for m in models}
        assert len(sums) == 1 and len(drifts) == 1
        ref = float((x - p).abs().double().sum()), float(c.abs().double().sum())
        assert next(iter(sums)) == pytest.approx(ref, rel=1e-12)
        del models


def test_two_threads_two_streams():
    P = need_gpu()
    models = [_model(P, s) for s in (3, 4)]
    data, want = [], []
    for i, m in enumerate(models):
        g = torch.Generator(device="cuda")
        g.manual_seed(10 + i)
        t = [torch.randn((CFG.n_video, CFG.hidden), generator=g, device="cuda") for _ in range(3)]
        data.append(t)
        want.append((m.l1_norms(*t), m.drift_signal(t[0], 0.5, t[1], torch.empty_like(t[0]))))
    torch.cuda.synchronize()
    bad = []

    def work(i):
        st = torch.cuda.Stream()
        x, p, c = data[i]
        with torch.cuda.stream(st):
            m_cur = torch.empty_like(x)
            for _ in range(50):
                got = (models[i].l1_norms(x, p, c), models[i].drift_signal(x, 0.5, p, m_cur))
                if got != want[i]:
                    bad.append((i, got, want[i]))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad, bad[:2]


@pytest.mark.parametrize("mode", ["acid", "easycache", "dicache"])
def test_loop_signals_of_nan_latents(mode):
    """A loop watches for its signals in the pinned slot: NaN signals arrive
    like any other, and the models of the 65th slot on, which copy theirs, and
    a repeated loop give the same trace."""
    P = need_gpu()
    models = [_model(P) for _ in range(65)]
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x0 = torch.randn((CFG.n_video, CFG.hidden), generator=g, device="cuda")
    for bad in (False, True):
        if bad:
            x0[3, 5] = float("nan")
        got = []
        for m in (models[0], models[0], models[64]):
            x = x0.clone()
            tr = m.denoise_loop(x, ai.sigmas(2), mode=mode, tau_low=0.05, tau_high=0.2, delta=0.01)
            got.append((tr.tobytes(), x.cpu().numpy().tobytes()))
            assert bool(x.isnan().any()) == bad
            if mode != "easycache":  # its first signal needs two computed steps
                assert bool(tr["s"][1] != tr["s"][1]) == bad
        assert got[0] == got[1] == got[2]


@pytest.mark.parametrize("blocks,heads", [(1, 4), (11, 8)])
def test_callers_own_loop_sees_the_same_signals(blocks, heads):
    """acid_drift_signal forms one pair of the modulation table, a loop all of
    it; TEMNI and signal are the same bits (11 blocks of hidden 512: the table
    is wide enough for another K split than the pair by itself would take)."""
    P = need_gpu()
    cfg = ai.TINY.replace(n_blocks=blocks, hidden=64 * heads, n_heads=heads, n_steps=4, n_video=40)
    m = P.Model(cfg, max_steps=4)
    g = torch.Generator(device="cuda")
    g.manual_seed(blocks)
    for tid, (_, shape) in enumerate(ai.manifest(cfg)):
        m.load_tensor(tid, torch.randn(shape, generator=g, device="cuda") * 0.05)
    x0 = torch.randn((cfg.n_video, cfg.hidden), generator=g, device="cuda")
    sig = ai.sigmas(4)
    kw = dict(mode="acid", tau_low=0.05, tau_high=0.2, delta=0.01)
    x = x0.clone()
    want = m.denoise_loop(x, sig, **kw)["s"].copy()
    prev, cur = torch.empty_like(x0), torch.empty_like(x0)
    for i in range(4):
        x = x0.clone()
        if i:
            m.denoise_loop(x, sig[: i + 1], **kw)  # x_i
        s = m.drift_signal(x, float(sig[i]), prev if i else None, cur)
        assert s == want[i] or (i == 0 and s != s), (i, s, want[i])
        prev, cur = cur, prev
