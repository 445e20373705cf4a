"""Advantages and word alignment where their kernels change path: batches at the size up to which a wave
remembers its group's entries."""
import numpy as np
import pytest
import torch

from oracle import mrl_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mrl():
    import paper_2605_07244_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("B,G,mode", [(63, 5, 1), (1025, 700, 2), (4096, 3, 1), (4097, 3, 1), (9001, 1200, 2)])
def test_advantages_remembered_and_scanned(mrl, B, G, mode):
    rng = np.random.default_rng(B)
    gid = rng.integers(-1, G + 1, B).astype(np.int32)            # interleaved; some ids outside [0, G)
    r = (rng.random(B) < 0.3).astype(np.float32)
    st, sc, own = ((rng.random(B) < p).astype(np.uint8) for p in (0.8, 0.7, 0.5))
    t = lambda a: torch.tensor(a, device="cuda")
    adv, mean, std, flags = mrl.group_advantages(t(r), t(gid), G, t(st), t(sc), t(own), mode=mode, mix_alpha=0.7)
    ok = (gid >= 0) & (gid < G)
    a_o, m_o, s_o, f_o = orc.group_advantages(r[ok].astype(np.float64), gid[ok], G, st[ok], sc[ok], own[ok], mode=mode, mix_alpha=0.7)
    got = adv.cpu().numpy()
    assert np.array_equal(flags.cpu().numpy(), f_o)
    assert np.allclose(mean.cpu().numpy(), m_o, rtol=1e-6, atol=1e-7) and np.allclose(std.cpu().numpy(), s_o, rtol=1e-6, atol=1e-7)
    # fp64 sums, one rounding to fp32 per value (two in mode 2)
    assert np.allclose(got[ok], a_o, rtol=3e-6, atol=1e-6)
    assert np.all(got[~ok] == 0) and np.all(got[sc == 0] == 0)
