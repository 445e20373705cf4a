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


def _cut(mrl, launch, rows, d, V, chunk_rows=0, tail_items=0):
    """(tiles of 384, 256, 128 along the tokens - dW: the vocabulary -, tiles of the last round, slices of each) of a launch."""
    c = mrl.gemm_cut(launch, rows, V, d, chunk_rows, 0, tail_items)
    return c["wide"], c["narrow"], c["half"], c["rest"], c["split"]


@pytest.mark.parametrize("N,scored,d,V", [
    (4096, 1, 128, 300),          # one row, two vocabulary tiles
    (4096, 257, 128, 2048),       # a column of 256 and one of 128, one whole band
    (2048, 700, 256, 8192),       # three columns of 256, 96 tiles: less than a round
    (2048, 1281, 128, 11000),     # three columns of 384 and one of 256, 43 vocabulary tiles (ragged last band), 172 tiles
    (4096, 4096, 128, 8300),      # every slot scored: ten columns of 384 and one of 256, 33 vocabulary tiles, 107 behind a whole round
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


@pytest.mark.parametrize("V", [120, 8192, 8200, 16400, 32800, 65536, 65600, 98400])
def test_partial_sums_in_batches(mrl, V):
    """A thread of the row epilogue adds every 64th of 2 ceil(V / 256) partial sums: 1, 1 and the next, 2 - 3, 4 - 5, a full batch of
    8, and 1 and 5 behind one."""
    H, W, y, mask = _head(130, 64, V, 129, V)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    rows = torch.nonzero(mask)[:, 0]
    Hs, Ws = util.to_f64(H[rows]), util.to_f64(W)
    want, want_lse = orc.token_logprobs(Hs, Ws, y[rows].cpu().numpy())
    want_ent = orc.token_entropy(Hs, Ws)
    for got, exact in ((logp, want), (lse, want_lse), (ent, want_ent)):
        assert np.max(np.abs(got[rows].cpu().numpy() - exact)) <= 1e-4


def _step(mrl, H, W, y, mask, dh_dtype, seed, chunk_rows=0, poison=False, hint=0):
    """One loss step of a single sequence (its tokens' advantages and traces random) and the same in float64.
    poison: the workspace holds NaN before the call."""
    g = torch.Generator("cuda").manual_seed(seed)
    N, d = H.shape
    V = W.shape[0]
    rows = torch.nonzero(mask)[:, 0]
    z = H[rows].double() @ W.double().t()
    lse = torch.logsumexp(z, 1)
    at = torch.arange(rows.numel(), device="cuda")
    lp = z[at, y[rows].long()] - lse
    behav = torch.zeros(N, device="cuda")
    behav[rows] = (lp + 0.05 * torch.randn(rows.numel(), device="cuda", generator=g)).float()
    cfg = mrl.LossConfig(kl_beta=0.0, dh_dtype=dh_dtype, chunk_rows=chunk_rows, scored_rows_hint=hint)
    ws = None
    if poison:
        code = mrl.F32 if H.dtype == torch.float32 else mrl.BF16
        ws = torch.full((mrl.grpo_loss_workspace(1, N, d, V, code, cfg),), 255, dtype=torch.uint8, device="cuda")
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, one(0.7, torch.float32), one(0, torch.int32), None, 1, N, 1, cfg, workspace=ws)
    torch.cuda.synchronize()
    w = torch.exp(lp - behav[rows].double())
    gr = torch.where(w <= 1.2, -0.7 * w, 0.0) / rows.numel()          # A > 0: clipped above 1.2
    dz = -gr[:, None] * torch.exp(z - lse[:, None])
    dz[at, y[rows].long()] += gr
    dH = torch.zeros((N, d), dtype=torch.float64, device="cuda")
    dH[rows] = dz @ W.double()
    return out, dH.cpu().numpy(), (dz.t() @ H[rows].double()).cpu().numpy()


@pytest.mark.parametrize("scored,d,V,dh_f32,cut", [
    (1, 256, 70, 0, (0, 0, 1, 1, 1)),                # one tile, a vocabulary shorter than a panel pair
    (300, 136, 1000, 1, (0, 0, 3, 3, 1)),            # three tiles of 128 over a padded width, too few panels to slice
    (255, 512, 9001, 0, (0, 0, 2, 4, 8)),            # four tiles of 128, eight slices
    (700, 1000, 16500, 1, (0, 0, 6, 24, 10)),        # float output from slices, a width that ends inside a tile
    (2500, 4096, 4200, 0, (6, 1, 0, 112, 2)),        # tiles of 384 and a row of tiles of 256, two slices
    (2500, 4096, 4200, 1, (6, 1, 0, 112, 2)),
    (4200, 4096, 5003, 0, (11, 0, 0, 176, 1)),       # 176 tiles of 384: more than half a round, left whole
    (4200, 4096, 5003, 1, (11, 0, 0, 176, 1)),
    (8300, 4096, 2000, 0, (21, 1, 0, 96, 2)),        # 352 tiles: a whole round and 96 of two slices
    (2500, 3080, 1000, 0, (0, 10, 0, 130, 1)),       # tiles of 256: whole
    (2500, 3080, 1000, 1, (0, 10, 0, 130, 1)),
    (8300, 264, 3001, 0, (0, 33, 0, 66, 3)),         # ... in slices, the last row of tiles with 108 tokens
    (5200, 3080, 8000, 0, (0, 21, 0, 17, 7)),        # ... a whole round and 17 of seven slices
])
def test_dh_tiles_and_slices(mrl, scored, d, V, dh_f32, cut):
    assert _cut(mrl, mrl.GEMM_DH, scored, d, V, -(-(scored + 37) // 256) * 256) == cut
    H, W, y, mask = _head(scored + 37, d, V, scored, scored)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.F32 if dh_f32 else mrl.BF16, scored)
    # bf16 operands (e, the scaled hidden rows, the output): 2^-9 each, the bar of the parity tests
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    assert torch.all(out["dH"][mask == 0] == 0)
    again, _, _ = _step(mrl, H, W, y, mask, mrl.F32 if dh_f32 else mrl.BF16, scored)
    assert torch.equal(out["dH"], again["dH"])


@pytest.mark.parametrize("N", [1, 63, 1025, 32768, 32769, 4096 * 1024, 4096 * 1024 + 5])
def test_compaction_paths(mrl, N):
    """One block, several blocks that add up the counts themselves, and the scan launch (above 4096 blocks of 1024
    slots); masked slots, target ids outside the vocabulary, zeros in every per-slot output of an unscored slot."""
    d, V = 8, 64
    g = torch.Generator("cuda").manual_seed(N)
    H = torch.randn((N, d), device="cuda", generator=g).bfloat16()
    W = torch.randn((V, d), device="cuda", generator=g).bfloat16()
    y = torch.randint(-2, V + 2, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = (torch.rand(N, device="cuda", generator=g) < 0.6).to(torch.uint8)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    torch.cuda.synchronize()
    ok = (mask == 1) & (y >= 0) & (y < V)
    z = H[ok].double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    want = z.gather(1, y[ok].long()[:, None])[:, 0] - want_lse
    want_ent = want_lse - (torch.softmax(z, 1) * z).sum(1)
    for got, ref in ((logp, want), (lse, want_lse), (ent, want_ent)):
        assert torch.all(got[~ok] == 0)
        # fp32 outputs of logits below 40: half a unit in the last place is 2e-6
        assert not ok.any() or float((got[ok].double() - ref).abs().max()) <= 2e-5


@pytest.mark.parametrize("N,d,V", [(1, 1, 3), (17, 3, 33), (40, 5, 16), (100, 64, 512), (530, 66, 515), (600, 71, 1000),
                                   (1000, 515, 1001), (1030, 520, 1100)])
def test_fp32_tiles_and_odd_widths(mrl, N, d, V):
    """fp32 products: K below, at and beside a multiple of 4 and of the 16-wide step, single tiles, ragged edges on every side.
    The 32 x 32 tile starts at 512 tiles (rows rounded up to 256): the forward product of 600 x 1000 outputs runs on it, 530 x
    515 (24 x 17 tiles) does not, and all three products of the last two shapes do."""
    g = torch.Generator("cuda").manual_seed(d)
    H = torch.randn((N, d), device="cuda", generator=g)
    W = 0.2 * torch.randn((V, d), device="cuda", generator=g)
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = (torch.rand(N, device="cuda", generator=g) < 0.9).to(torch.uint8)
    mask[0] = 1
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.F32, 5)
    ok = mask == 1
    z = H[ok].double() @ W.double().t()
    want = z.gather(1, y[ok].long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    # at most 1100 fp32 terms per sum: sqrt(1100) * 2^-24 relative, a hundred times below the bars
    assert float((out["logp"][ok].double() - want).abs().max()) <= util.F32_LOGP_TOL
    for name, got, ref in (("dH", out["dH"], dH), ("dW", out["dW"], dW)):
        assert util.rel_fro(util.to_f64(got), ref) <= 1e-5 or np.linalg.norm(ref) < 1e-12, name
    assert torch.all(out["dH"][~ok] == 0)


@pytest.mark.parametrize("scored,d,V", [(1, 128, 100), (64, 136, 129), (65, 256, 256), (200, 1536, 5000), (256, 128, 8321)])
def test_forward_of_few_rows(mrl, scored, d, V):
    """Passes of at most 256 rows: vocabularies that end in the first or the second half of a pair of 128-wide tiles, token
    counts around a wave's 64, log-probs, entropy and (through the stash) both gradients."""
    H, W, y, mask = _head(scored, d, V, scored, d + V)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, V)
    torch.cuda.synchronize()
    z = H.double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    want = z.gather(1, y.long()[:, None])[:, 0] - want_lse
    # fp32 sums of at most 8321 exponentials and 1536 products: far below the bar
    assert float((logp.double() - want).abs().max()) <= 1e-4 and float((lse.double() - want_lse).abs().max()) <= 1e-4
    assert float((ent.double() - (want_lse - (torch.softmax(z, 1) * z).sum(1))).abs().max()) <= 1e-4
    assert torch.equal(out["logp"], logp)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)


@pytest.mark.parametrize("N,d,V", [(1, 72, 4000), (70, 200, 3000), (129, 136, 5000), (256, 448, 8200)])
def test_forward_of_few_rows_from_any_column(mrl, N, d, V):
    """Passes of at most 256 rows whose tiles start at different columns: the walk goes round behind the zero-padded end of K
    (all of the head copied, or its last 128 columns), waves with and without tokens."""
    H, W, y, mask = _head(N, d, V, N, N + d)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.F32, V, poison=True)
    torch.cuda.synchronize()
    z = H.double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    # fp32 sums of at most 8200 exponentials and 448 products: far below the bar
    assert float((logp.double() - (z.gather(1, y.long()[:, None])[:, 0] - want_lse)).abs().max()) <= 1e-4
    assert float((ent.double() - (want_lse - (torch.softmax(z, 1) * z).sum(1))).abs().max()) <= 1e-4
    assert torch.equal(out["logp"], logp)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)


@pytest.mark.parametrize("scored,d,V", [(257, 128, 700), (320, 200, 2500), (384, 256, 6000), (385, 128, 1000), (1921, 136, 4400)])
def test_forward_half_columns(mrl, scored, d, V):
    """A last column of at most 128 tokens (one, those of one wave, all, one too many) behind one or seven whole ones, over one and
    several bands of tile rows: log-probs, entropy and both gradients."""
    H, W, y, mask = _head(scored + 40, d, V, scored, scored + d)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.F32, V, poison=True)
    torch.cuda.synchronize()
    ok = mask == 1
    z = H[ok].double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    want = z.gather(1, y[ok].long()[:, None])[:, 0] - want_lse
    # fp32 sums of at most 6000 exponentials and 256 products: far below the bar
    assert float((logp[ok].double() - want).abs().max()) <= 1e-4 and float((lse[ok].double() - want_lse).abs().max()) <= 1e-4
    assert float((ent[ok].double() - (want_lse - (torch.softmax(z, 1) * z).sum(1))).abs().max()) <= 1e-4
    assert torch.equal(out["logp"], logp)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)


@pytest.mark.parametrize("N,d,V", [(100, 120, 700), (300, 136, 700), (4096, 200, 900), (4200, 200, 900), (4200, 192, 900)])
def test_padded_widths(mrl, N, d, V):
    """Widths beside a multiple of 128: a head narrower than a panel pair, the head's zero-padded tail next to its own rows
    (up to 4096 rows, and above for rows of whole lines), a padded copy of all of it."""
    H, W, y, mask = _head(N, d, V, N - 3, d)
    logp, lse = mrl.token_logprobs(H, W, y, mask)
    torch.cuda.synchronize()
    ok = mask == 1
    z = H[ok].double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    assert float((lse[ok].double() - want_lse).abs().max()) <= 1e-4
    assert float((logp[ok].double() - (z.gather(1, y[ok].long()[:, None])[:, 0] - want_lse)).abs().max()) <= 1e-4


@pytest.mark.parametrize("scored", [1, 129, 327, 700, 1030])
def test_dw_tail_slices_without_panels(mrl, scored):
    """The tail of this head is planned as 8 slices; 2, 4, 6, 12 and 18 panels fill 1, 2, 3, 6 and 5 of them.  The others store
    nothing and are not read: the scratch holds NaN before.  (A pass that can hold 1280 rows, which is what the launch goes by.)"""
    d, V = 1024, 16405
    assert mrl.dw_tail_plan(V, d)["split"] == 8 and mrl.dw_few_rows() < 1280 and _cut(mrl, mrl.GEMM_DW, scored, d, V, 1280) == (0, 65, 0, 4, 8)
    H, W, y, mask = _head(scored + 3, d, V, scored, scored)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, scored, chunk_rows=1280, poison=True)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)


@pytest.mark.parametrize("N,d,V", [(100, 64, 512), (1000, 515, 1001)])
def test_fp32_one_gradient_alone(mrl, N, d, V):
    """dH or dW alone: the launches of their own, on 16 x 16 and 32 x 32 tiles, give the bits of the call for both (which
    shares a launch at the smaller shape)."""
    g = torch.Generator("cuda").manual_seed(V)
    H, W = torch.randn((N, d), device="cuda", generator=g), 0.2 * torch.randn((V, d), device="cuda", generator=g)
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = torch.ones(N, dtype=torch.uint8, device="cuda")
    behav = torch.full((N,), -6.0, device="cuda")
    adv, gid = torch.tensor([0.5], device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    cfg = mrl.LossConfig(kl_beta=0.0, dh_dtype=mrl.F32)
    call = lambda **kw: mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, adv, gid, None, 1, N, 1, cfg, **kw)
    both, only_h, only_w = call(), call(want_dW=False), call(want_dH=False)
    torch.cuda.synchronize()
    assert torch.equal(both["dH"], only_h["dH"]) and torch.equal(both["dW"], only_w["dW"])
    assert only_h["dW"] is None and only_w["dH"] is None and float(both["dH"].abs().max()) > 0


@pytest.mark.parametrize("N,d,V", [(4200, 192, 900), (4200, 200, 900), (300, 136, 700)])
def test_gradients_of_padded_widths(mrl, N, d, V):
    """Both gradients beside the head's zero-padded tail (rows of whole lines above 4096 rows, any rows below) and its full copy."""
    H, W, y, mask = _head(N, d, V, N - 5, d)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, d, poison=True)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)


@pytest.mark.parametrize("N,scored,chunk_rows", [
    (16500, 16500, 0),            # forward parts of 16384 and 256 rows, the second with 116 valid ones
    (16500, 9000, 0),             # ... and with none
    (16640, 16640, 0),            # ... and with all 256
    (700, 650, 256),              # three passes of at most 256 rows, the last with 138
])
def test_few_rows_behind_others(mrl, N, scored, chunk_rows):
    """Up to 256 rows as the last part of a larger pass, on the large tile or a half column of it (rows, partial sums and stash at
    an offset, the partials' stride that of the pass), and passes of 256 rows, on the forward kernel for few rows."""
    d, V = 64, 600
    H, W, y, mask = _head(N, d, V, scored, N + scored)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, scored, chunk_rows=chunk_rows, poison=True)
    logp, lse, ent = mrl.token_scores(H, W, y, mask)
    torch.cuda.synchronize()
    ok = mask == 1
    z = H[ok].double() @ W.double().t()
    want_lse = torch.logsumexp(z, 1)
    want = z.gather(1, y[ok].long()[:, None])[:, 0] - want_lse
    want_ent = want_lse - (torch.softmax(z, 1) * z).sum(1)
    # fp32 sums of 600 exponentials and 64 products: far below the bar
    for got, ref in ((logp, want), (lse, want_lse), (ent, want_ent), (out["logp"], want)):
        assert float((got[ok].double() - ref).abs().max()) <= 1e-4 and torch.all(got[~ok] == 0)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    assert torch.all(out["dH"][~ok] == 0)


@pytest.mark.parametrize("scored,d,V,cut", [(1100, 8192, 21000, (3, 0, 0, 96, 5)), (1100, 8192, 40003, (3, 0, 0, 96, 8))])
def test_dh_slices_in_two_rounds(mrl, scored, d, V, cut):
    """96 tiles of five and of eight slices: more items than compute units, in two and in three rounds."""
    assert _cut(mrl, mrl.GEMM_DH, scored, d, V, -(-(scored + 5) // 256) * 256) == cut and cut[3] * cut[4] > 256
    H, W, y, mask = _head(scored + 5, d, V, scored, 9)
    rows = torch.nonzero(mask)[:, 0]
    z = H[rows].double() @ W.double().t()
    lse = torch.logsumexp(z, 1)
    at = torch.arange(scored, device="cuda")
    lp = z[at, y[rows].long()] - lse
    behav = torch.zeros(scored + 5, device="cuda")
    behav[rows] = lp.float()
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, one(0.7, torch.float32), one(0, torch.int32), None, 1, scored + 5, 1,
                                mrl.LossConfig(kl_beta=0.0), want_dW=False)
    gr = -0.7 * torch.exp(lp - behav[rows].double()) / scored
    dz = -gr[:, None] * torch.exp(z - lse[:, None])
    dz[at, y[rows].long()] += gr
    want = torch.zeros((scored + 5, d), dtype=torch.float64, device="cuda")
    want[rows] = dz @ W.double()
    util.check_gradient("dH", util.to_f64(out["dH"]), want.cpu().numpy())
    assert torch.all(out["dH"][mask == 0] == 0)


@pytest.mark.parametrize("level", [1, 2])
def test_fp32_response_ratio_over_passes(mrl, level):
    """Three fp32 passes, swept last to first for the log-probs: the target logits of all rows come with the first one swept."""
    B, T, d, V = 40, 130, 24, 90
    N = B * T
    g = torch.Generator("cuda").manual_seed(level)
    H, W = torch.randn((N, d), device="cuda", generator=g), 0.2 * torch.randn((V, d), device="cuda", generator=g)
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = (torch.rand(N, device="cuda", generator=g) < 0.95).to(torch.uint8)
    adv, gid = torch.randn(B, device="cuda", generator=g), torch.zeros(B, dtype=torch.int32, device="cuda")
    z = H.double() @ W.double().t()
    lp = z.gather(1, y.long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    behav = (lp + 0.01 * (torch.rand(N, device="cuda", generator=g) - 0.5)).float()      # ratios inside the clip range
    out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, adv, gid, None, B, T, 1,
                                mrl.LossConfig(kl_beta=0.0, dh_dtype=mrl.F32, ratio_level=level))
    m = mask.double()
    L = m.view(B, T).sum(1)
    expo = ((lp - behav.double()) * m).view(B, T).sum(1) / (L if level == 2 else 1.0)
    assert float(expo.abs().max()) < 0.18
    gr = (-(torch.exp(expo) * adv.double()) / (B * (L if level == 2 else 1.0))).repeat_interleave(T) * m
    dz = -gr[:, None] * torch.softmax(z, 1)
    dz[torch.arange(N, device="cuda"), y.long()] += gr
    for name, got, want in (("logp", out["logp"], lp * m), ("dH", out["dH"], dz @ W.double()), ("dW", out["dW"], dz.t() @ H.double())):
        # fp32 sums of 24, 90 and 4940 terms
        error, size = float((got.double() - want).norm()), float(want.norm())
        assert error <= 1e-5 * size, (name, error, size)


@pytest.mark.parametrize("N,scored,d,V", [
    (820, 800, 512, 5003),        # a last half column in the long pass; 40 vocabulary tiles of 128, eight K chunks
    (1020, 1000, 712, 2057),      # a padded width, the last column a whole tile
    (533, 513, 4096, 1300),       # power-of-two rows, 64 K chunks; one row in the last column
    (700, 100, 4096, 50001),      # ... and tiles enough that they start one after another
    (700, 129, 2048, 100003),     # ... and one row too many for that
])
def test_scores_do_not_depend_on_the_pass(mrl, N, scored, d, V):
    """Every forward kernel adds a logit's products in the same order: the bits of a token's scores are those of a long pass, of
    passes of 256 rows (a workspace that holds no longer one, or chunk_rows) and of a call of a few slots."""
    H, W, y, mask = _head(N, d, V, scored, V)
    want = mrl.token_scores(H, W, y, mask)
    # 16 KB more than 256 slots take hold the arrays by slot, and no pass of 512 rows
    small = int(mrl.lib().mrl_token_scores_workspace(256, d, V, mrl.BF16)) + 16384
    assert small < int(mrl.lib().mrl_token_scores_workspace(512, d, V, mrl.BF16))
    passes = mrl.token_scores(H, W, y, mask, workspace=torch.empty(small, dtype=torch.uint8, device="cuda"))
    alone = [mrl.token_scores(H[r:r + 190], W, y[r:r + 190], mask[r:r + 190]) for r in range(0, N, 190)]
    torch.cuda.synchronize()
    for k in range(3):
        assert torch.equal(passes[k], want[k])
        assert torch.equal(torch.cat([a[k] for a in alone]), want[k])
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    for chunk_rows in (0, 256):
        out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, torch.zeros(N, device="cuda"), None, one(0.7, torch.float32), one(0, torch.int32),
                                    None, 1, N, 1, mrl.LossConfig(kl_beta=0.0, chunk_rows=chunk_rows), want_dW=False)
        assert torch.equal(out["logp"], want[0])


@pytest.mark.parametrize("scored,d,V", [(200, 128, 129), (700, 256, 8), (1500, 240, 329), (600, 512, 2057)])
def test_dw_beside_the_pad_columns(mrl, scored, d, V):
    """Vocabularies that end in the first chunk of a tile, a chunk behind a 128-wide half and inside one: the launch reads other
    columns in the pad's place, and the rows of dW do not see it."""
    H, W, y, mask = _head(scored + 3, d, V, scored, V)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, V, poison=True)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)


@pytest.mark.parametrize("N,scored,d,V,shift", [
    (1, 1, 8, 2, 0),              # one row, one tile of which two ids and eight columns are there
    (300, 129, 96, 127, 0),       # whole-line rows, a tile short of one id; two panel pairs
    (300, 128, 136, 129, 1),      # rows that straddle lines, at 4-byte alignment; two tile rows
    (1024, 1000, 264, 700, 0),    # two tile columns, the second of 8
    (1024, 1024, 512, 5000, 3),   # whole-line widths at 4-byte alignment; 40 x 2 tiles
    (900, 0, 128, 300, 0),        # no rows: zeros, or dW untouched
])
def test_dw_of_few_rows(mrl, N, scored, d, V, shift):
    """The dW launch for at most 1024 rows, overwriting and accumulating into earlier values, dW at any float address."""
    H, W, y, mask = _head(N, d, V, scored, N + d)
    if scored > 0:
        _, _, want = _step(mrl, H, W, y, mask, mrl.F32, V, poison=True)
    else:
        want = np.zeros((V, d))
    g = torch.Generator("cuda").manual_seed(V)
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    for accumulate in (0, 1):
        # the values around dW belong to others
        buf = torch.randn(V * d + 64, device="cuda", generator=g) * 1e-3
        dW = buf[32 + shift:32 + shift + V * d].view(V, d)
        before = buf.clone()
        cfg = mrl.LossConfig(kl_beta=0.0, dh_dtype=mrl.F32, accumulate_dw=accumulate)
        ws = torch.full((mrl.grpo_loss_workspace(1, N, d, V, mrl.BF16, cfg),), 255, dtype=torch.uint8, device="cuda")
        behav = _behaviour(H, W, y, mask, V)
        mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, one(0.7, torch.float32), one(0, torch.int32), None, 1, N, 1, cfg,
                              out_dW=dW, workspace=ws)
        torch.cuda.synchronize()
        old = before[32 + shift:32 + shift + V * d].view(V, d)
        got = util.to_f64(dW) - (util.to_f64(old) if accumulate else 0.0)
        if scored > 0:
            # accumulating: one rounding of a sum of at most 5e-3 + |dW| more than the oracle's
            slack = 2.0 ** -24 * (5e-3 + np.abs(want).max()) * accumulate
            assert np.abs(got - want).max() <= 1e-2 * np.abs(want).max() + slack
            assert util.rel_fro(got, want) <= util.REL_TOL + slack * np.sqrt(want.size) / np.linalg.norm(want)
        else:
            assert np.all(got == 0)
        assert torch.equal(buf[:32 + shift], before[:32 + shift]) and torch.equal(buf[32 + shift + V * d:], before[32 + shift + V * d:])


def _behaviour(H, W, y, mask, seed):
    """The behaviour trace that _step draws."""
    g = torch.Generator("cuda").manual_seed(seed)
    rows = torch.nonzero(mask)[:, 0]
    z = H[rows].double() @ W.double().t()
    lp = z[torch.arange(rows.numel(), device="cuda"), y[rows].long()] - torch.logsumexp(z, 1)
    behav = torch.zeros(H.shape[0], device="cuda")
    behav[rows] = (lp + 0.05 * torch.randn(rows.numel(), device="cuda", generator=g)).float()
    return behav


@pytest.mark.parametrize("scored", [1025, 1400])
def test_dw_k_split_tail_above_the_few_rows(mrl, scored):
    """The large dW launch with its ragged last tile rows cut into eight K slices: more than 1024 rows, a second pass that
    adds into the first's result, poisoned scratch."""
    d, V = 1536, 11000
    assert mrl.dw_tail_plan(V, d)["split"] == 8 and mrl.dw_few_rows() == 1024
    assert all(_cut(mrl, mrl.GEMM_DW, 1025, d, V, chunk) == (0, 43, 0, 18, 8) for chunk in (1280, 1536))
    H, W, y, mask = _head(1500, d, V, scored, scored)
    out, _, dW = _step(mrl, H, W, y, mask, mrl.BF16, V, poison=True)
    again, _, _ = _step(mrl, H, W, y, mask, mrl.BF16, V, poison=True)
    two, _, _ = _step(mrl, H, W, y, mask, mrl.BF16, V, chunk_rows=1280, poison=True)
    assert torch.equal(out["dW"], again["dW"])
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    util.check_gradient("dW", util.to_f64(two["dW"]), dW)


@pytest.mark.parametrize("scored,chunk_rows", [(900, 0), (900, 4096), (1500, 1280)])
def test_hint_and_dw_launch(mrl, scored, chunk_rows):
    """The hint chooses the dW launch for few rows inside a pass that could hold more (and, as 300, more than it says): dW to
    rounding and everything else bit for bit what the call without a hint gives.  In the last case the second of two passes takes
    that launch, by what the hint leaves to it."""
    d, V = 1536, 11000
    assert mrl.dw_tail_plan(V, d)["split"] == 8 and mrl.dw_few_rows() == 1024
    H, W, y, mask = _head(1530, d, V, scored, scored)
    out, _, dW = _step(mrl, H, W, y, mask, mrl.BF16, V, chunk_rows=chunk_rows, poison=True)
    stats = mrl.read_stats(out["stats"])
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    for hint in (scored, 300) if scored < 1024 else (scored,):
        got, _, _ = _step(mrl, H, W, y, mask, mrl.BF16, V, chunk_rows=chunk_rows, poison=True, hint=hint)
        assert torch.equal(got["logp"], out["logp"]) and torch.equal(got["dH"], out["dH"])
        assert mrl.read_stats(got["stats"]) == stats and stats["n_unprocessed_rows"] == 0
        # fp32 sums of at most 2000 products in two orders: 2^-24 * sqrt(2000) of the largest sum of absolute terms
        assert float((got["dW"] - out["dW"]).abs().max()) <= 1e-5 * float(out["dW"].abs().max())


@pytest.mark.parametrize("scored,chunk_rows,d,V,cuts", [
    (1500, 4096, 136, 1000, ((3, 0, 0, 3, 3), (0, 4, 0, 0, 1))),         # tiles of 384 in three slices without the hint, whole ones of 256 with it
    (2000, 4096, 520, 9999, ((27, 0, 0, 81, 3), (0, 40, 0, 0, 1))),
])
def test_hint_above_the_few_rows(mrl, scored, chunk_rows, d, V, cuts):
    """The hint also chooses between the larger and the smaller tiles of dW: dW to rounding, everything else bit for bit."""
    for expected, cut in zip((chunk_rows, scored), cuts):
        c = mrl.gemm_cut(mrl.GEMM_DW, scored, V, d, chunk_rows, expected)
        assert (c["wide"], c["narrow"], c["half"], c["rest"], c["split"]) == cut
    H, W, y, mask = _head(chunk_rows, d, V, scored, scored)
    out, _, dW = _step(mrl, H, W, y, mask, mrl.BF16, V, chunk_rows=chunk_rows, poison=True)
    got, _, _ = _step(mrl, H, W, y, mask, mrl.BF16, V, chunk_rows=chunk_rows, poison=True, hint=scored)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    assert torch.equal(got["logp"], out["logp"]) and torch.equal(got["dH"], out["dH"])
    assert mrl.read_stats(got["stats"]) == mrl.read_stats(out["stats"])
    # fp32 sums of at most 2000 products in two orders: 2^-24 * sqrt(2000) of the largest sum of absolute terms
    assert float((got["dW"] - out["dW"]).abs().max()) <= 1e-5 * float(out["dW"].abs().max())


@pytest.mark.parametrize("N,scored,V,chunk_rows", [
    (1, 1, 2, 0), (40, 17, 64, 0), (300, 300, 65, 256), (33, 33, 512, 0), (33, 33, 513, 0), (500, 260, 2047, 256), (272, 257, 2048, 0), (272, 257, 2049, 0),
])
def test_fp32_rows_in_one_launch(mrl, N, scored, V, chunk_rows):
    """fp32 loss calls around the vocabulary up to which a row's log-sum-exp, loss terms and dz share a launch: rows beside a
    multiple of its 16 per block, a second pass with one row or a part of them, poisoned scratch; gradients and statistics."""
    d = 40
    H, W, y, mask = _head(N, d, V, scored, N + V)
    H, W = H.float(), 10 * W.float()
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.F32, V, chunk_rows=chunk_rows, poison=True)
    rows = torch.nonzero(mask)[:, 0]
    z = H[rows].double() @ W.double().t()
    lp = z.gather(1, y[rows].long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    # fp32 sums of at most 2049 terms: 2^-24 * sqrt(2049) relative, times the depth of the chain
    assert float((out["logp"][rows].double() - lp).abs().max()) <= 2e-5
    assert util.rel_fro(util.to_f64(out["dH"]), dH) <= 2e-5 and util.rel_fro(util.to_f64(out["dW"]), dW) <= 2e-5
    st = mrl.read_stats(out["stats"])
    w = torch.exp(lp - _behaviour(H, W, y, mask, V)[rows].double())
    loss = -float(torch.minimum(0.7 * w, 0.7 * w.clamp(0.8, 1.2)).mean())
    assert abs(st["loss_pg"] - loss) <= 1e-5 * abs(loss) and st["n_scored_tokens"] == scored
    assert abs(st["mean_ratio"] - float(w.mean())) <= 2e-5 and abs(st["max_ratio"] - float(w.max())) <= 5e-5


@pytest.mark.parametrize("B,T,extra", [(2048, 1, 8), (1, 2048, 1), (7, 292, 8), (32, 64, 2)])
def test_prep_inside_the_row_preparation(mrl, B, T, extra):
    """Up to 2048 slots the mask is compacted by the row preparation's own blocks.  The same call with `extra` empty auxiliary
    sequences behind it has more slots and a preparation launch: the same bits.  Bad targets and group ids in both."""
    d, V, G = 72, 300, 3 if B > 1 else 1
    N, M = B * T, (B + extra) * T
    assert N <= 2048 < M
    g = torch.Generator("cuda").manual_seed(B)
    H = torch.randn((M, d), device="cuda", generator=g).bfloat16()
    W = (0.1 * torch.randn((V, d), device="cuda", generator=g)).bfloat16()
    y = torch.randint(0, V, (M,), device="cuda", generator=g, dtype=torch.int32)
    mask = (torch.rand(M, device="cuda", generator=g) < 0.6).to(torch.uint8)
    mask[N:] = 0
    y[torch.randperm(N, device="cuda", generator=g)[:5]] = V
    behav = torch.randn(M, device="cuda", generator=g) * 0.1 - 6
    adv = torch.randn(B + extra, device="cuda", generator=g)
    group = torch.randint(0, G, (B + extra,), device="cuda", generator=g, dtype=torch.int32)
    if B > 1:
        group[1] = G
    kind = torch.zeros(B + extra, dtype=torch.uint8, device="cuda")
    kind[B:] = 1
    cfg = mrl.LossConfig(kl_beta=0.0, dh_dtype=mrl.F32)

    def call(b):
        n = b * T
        ws = torch.full((mrl.grpo_loss_workspace(b, T, d, V, mrl.BF16, cfg),), 255, dtype=torch.uint8, device="cuda")
        out = mrl.grpo_loss_fwd_bwd(H[:n], W, y[:n], mask[:n], behav[:n], None, adv[:b], group[:b], kind[:b], b, T, G, cfg,
                                    workspace=ws)
        scores = mrl.token_scores(H[:n], W, y[:n], mask[:n])
        torch.cuda.synchronize()
        return out, mrl.read_stats(out["stats"]), scores

    (a, sa, ca), (b, sb, cb) = call(B), call(B + extra)
    assert sa == sb and sa["n_bad_targets"] > 0 and sa["n_scored_tokens"] > 0
    assert torch.equal(a["logp"], b["logp"][:N]) and torch.equal(a["dH"], b["dH"][:N])
    assert torch.equal(a["dW"], b["dW"])
    assert all(torch.equal(p, q[:N]) and torch.all(q[N:] == 0) for p, q in zip(ca, cb))
    assert torch.all(a["logp"][mask[:N] == 0] == 0) and torch.all(a["dH"][mask[:N] == 0] == 0)


@pytest.mark.parametrize("scored,d,V,chunk_rows,fwd,dh,dw", [
    (600, 128, 32005, 1280, (1, 1, 0, 252, 1), (0, 0, 5, 5, 31), (0, 126, 0, 0, 1)),      # forward: a column of 384 and one of 256, a ragged last row of W
    (700, 136, 32000, 0, (2, 0, 0, 250, 1), (0, 0, 6, 6, 31), None),                      # two columns of 384, the second with 316 tokens; a padded width
    (1152, 256, 30001, 2048, (3, 0, 0, 98, 1), (0, 0, 9, 9, 28), (0, 118, 0, 0, 1)),      # three whole columns of 384
    (300, 1032, 32005, 0, (0, 2, 0, 252, 1), (0, 0, 3, 15, 17), None),                    # 44 tokens in a last column of 256, a round nearly full
    (4200, 1032, 24000, 0, (10, 1, 1, 104, 1), (0, 17, 0, 85, 3), (0, 94, 0, 30, 2)),     # a last column of 384 as one of 256 and one of 128
    (2000, 256, 40003, 0, (0, 8, 0, 232, 1), (0, 0, 16, 16, 16), (0, 157, 0, 0, 1)),
    (2000, 136, 1000, 0, (0, 8, 0, 32, 1), (0, 0, 16, 16, 1), (3, 0, 0, 3, 4)),           # dW: three tiles of four slices
    (2000, 264, 40003, 1280, (0, 5, 0, 17, 1), (0, 0, 10, 20, 12), (105, 0, 0, 210, 1)),  # dW: tiles of 384 left whole, a second pass that adds into the first's result
    (2000, 3080, 9999, 0, (4, 2, 0, 240, 1), (4, 2, 0, 78, 3), (27, 0, 0, 95, 2)),        # dW: a whole round, and 95 tiles of two slices
    (3200, 3080, 9999, 1792, (4, 1, 0, 200, 1), (4, 1, 0, 65, 3), (27, 0, 0, 95, 2)),      # ... twice
    (3500, 2056, 21000, 0, (0, 14, 0, 138, 1), (0, 14, 0, 126, 2), (55, 0, 0, 239, 1)),   # dW: 239 tiles behind a whole round
])
def test_tiles_of_384(mrl, scored, d, V, chunk_rows, fwd, dh, dw):
    """The large tiles of the three products: whole, ragged and in slices; the log-probs have the bits that a pass of few rows gives.
    The cuts are those of the first pass."""
    N = scored + 21
    chunk = chunk_rows or -(-N // 256) * 256
    for launch, cut in ((mrl.GEMM_FWD, fwd), (mrl.GEMM_DH, dh), (mrl.GEMM_DW, dw)):
        assert _cut(mrl, launch, min(scored, chunk), d, V, chunk) == (cut or (0, 0, 0, 0, 0)), launch
    H, W, y, mask = _head(N, d, V, scored, scored + d)
    out, dH, dW = _step(mrl, H, W, y, mask, mrl.BF16, d, chunk_rows=chunk_rows, poison=True)
    util.check_gradient("dH", util.to_f64(out["dH"]), dH)
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    assert torch.all(out["dH"][mask == 0] == 0) and torch.all(out["logp"][mask == 0] == 0)
    again, _, _ = _step(mrl, H, W, y, mask, mrl.BF16, d, chunk_rows=chunk_rows, poison=True)
    assert all(torch.equal(out[k], again[k]) for k in ("logp", "dH", "dW"))
    for first in (0, N - 200):
        few, _ = mrl.token_logprobs(H[first:first + 200], W, y[first:first + 200], mask[first:first + 200])
        assert torch.equal(few, out["logp"][first:first + 200])


def test_workspace_without_room_for_all_partial_tiles(mrl):
    """A loss call takes a workspace whose end holds two thirds of the partial tiles (what it held when they were 256 x 256), and none
    smaller: the tiles of the last rounds are cut into fewer slices."""
    scored, d, V = 900, 1024, 30000
    H, W, y, mask = _head(scored, d, V, scored, 3)
    cfg = mrl.LossConfig(kl_beta=0.0, chunk_rows=1024)
    full = mrl.grpo_loss_workspace(1, scored, d, V, mrl.BF16, cfg)
    items = 256 + min(768, d * (-(-V // 256) * 256 + 64) * 2 // 4 // (256 * 256 * 4))
    least = full - items * 128 * 256 * 4
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    call = lambda n: mrl.grpo_loss_fwd_bwd(H, W, y, mask, torch.full((scored,), -10.0, device="cuda"), None, one(0.7, torch.float32),
                                           one(0, torch.int32), None, 1, scored, 1, cfg, workspace=torch.full((n,), 255, dtype=torch.uint8, device="cuda"))
    want, got = call(full), call(least)
    torch.cuda.synchronize()
    assert torch.equal(got["logp"], want["logp"])
    # dH is a bf16 result of fp32 sums in another order: neighbours at most; dW's order does not change
    assert float((got["dH"].float() - want["dH"].float()).abs().max()) <= 2 ** -7 * float(want["dH"].float().abs().max())
    util.check_gradient("dW", util.to_f64(got["dW"]), util.to_f64(want["dW"]))
    with pytest.raises(RuntimeError):
        call(least - 256)


@pytest.mark.parametrize("scored,d,V,full,least", [
    (2500, 136, 14001, (37, 0, 0, 37, 5), (37, 0, 0, 37, 4)),          # tiles of 384: fewer slices
    (1100, 2304, 7424, (0, 29, 0, 45, 5), (0, 29, 0, 45, 5)),          # tiles of 256: 225 items, smaller ones, as before
])
def test_dw_slices_in_the_least_workspace(mrl, scored, d, V, full, least):
    """dW's partial tiles, above the rows that have a launch without any, in the smallest workspace that a pass takes: nothing
    is written behind it, and dW is that of the full one to rounding."""
    assert scored > mrl.dw_few_rows()
    chunk = -(-scored // 256) * 256
    items = mrl.gemm_cut(mrl.GEMM_DW, scored, V, d, chunk)["tail_items"]
    H, W, y, mask = _head(scored, d, V, scored, 5)
    cfg = mrl.LossConfig(kl_beta=0.0, chunk_rows=chunk)
    size = mrl.grpo_loss_workspace(1, scored, d, V, mrl.BF16, cfg)
    small = size - items * 128 * 256 * 4
    assert _cut(mrl, mrl.GEMM_DW, scored, d, V, chunk) == full and _cut(mrl, mrl.GEMM_DW, scored, d, V, chunk, items * 2 // 3) == least
    _, _, dW = _step(mrl, H, W, y, mask, mrl.BF16, 7, chunk_rows=chunk)
    behav = _behaviour(H, W, y, mask, 7)
    one = lambda v, t: torch.tensor([v], dtype=t, device="cuda")
    buf = torch.full((small + 4096,), 255, dtype=torch.uint8, device="cuda")
    out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, one(0.7, torch.float32), one(0, torch.int32), None, 1, scored, 1, cfg, workspace=buf[:small])
    torch.cuda.synchronize()
    util.check_gradient("dW", util.to_f64(out["dW"]), dW)
    assert torch.all(buf[small:] == 255)
