"""The GEMM launches' distribution of tiles over workgroups: scored-row counts and vocabularies whose
tile counts leave ragged bands, incomplete rounds of 256 tiles and columns beyond the scored rows."""
import numpy as np
import pytest
import torch

from oracle import mrl_oracle as orc
from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mrl():
    import paper_2605_07244_amd as m
    m.lib()
    return m


def _head(N, d, V, scored, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    H = torch.randn((N, d), device="cuda", generator=g).bfloat16()
    W = (0.02 * torch.randn((V, d), device="cuda", generator=g)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = torch.zeros(N, dtype=torch.uint8, device="cuda")
    mask[torch.randperm(N, device="cuda", generator=g)[:scored]] = 1
    return H, W, y, mask


@pytest.mark.parametrize("N,scored,d,V", [
    (4096, 1, 128, 300),          # one row, two vocabulary tiles
    (4096, 257, 128, 2048),       # two tile columns of sixteen, one whole band
    (2048, 700, 256, 8192),       # three of eight columns, 96 tiles: less than a round
    (2048, 1281, 128, 11000),     # six columns, 43 vocabulary tiles (ragged last band), 258 tiles
    (4096, 4096, 128, 8300),      # every slot scored: sixteen columns, 33 vocabulary tiles
])
def test_forward_tiles_cover_scored_rows(mrl, N, scored, d, V):
    H, W, y, mask = _head(N, d, V, scored, N + scored)
    logp, lse = mrl.token_logprobs(H, W, y, mask)
    torch.cuda.synchronize()
    rows = torch.nonzero(mask)[:, 0]
    want, want_lse = orc.token_logprobs(util.to_f64(H[rows]), util.to_f64(W), y[rows].cpu().numpy())
    # fp32 sums of bf16 products: 2^-24 * sqrt(V) relative on the exponential sums, far below the bar
    assert np.max(np.abs(logp[rows].cpu().numpy() - want)) <= 1e-4
    assert np.max(np.abs(lse[rows].cpu().numpy() - want_lse)) <= 1e-4
    assert torch.all(logp[mask == 0] == 0) and torch.all(lse[mask == 0] == 0)
