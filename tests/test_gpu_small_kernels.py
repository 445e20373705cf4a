"""Advantages, word alignment and the aggregation weights where their kernels change path: batches at the size up to
which a wave remembers its group's entries, alignment segments, group counts in LDS and in global memory."""
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


@pytest.mark.parametrize("B,G,mode", [(63, 5, 1), (1025, 700, 2), (4096, 3, 1), (4097, 3, 1), (9001, 1200, 2), (4353, 1, 0), (20000, 5, 2)])
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


@pytest.mark.parametrize("B,S_src,S_tgt,one_word", [(3, 1, 1, True), (5, 257, 700, True), (2, 8192, 8193, False), (2, 9100, 10000, False),
                                                     (7, 63, 65, False), (6, 64, 64, True), (9, 65, 200, True), (6, 256, 256, True),
                                                     (40, 230, 256, False), (5, 256, 257, False), (5, 257, 250, True)])
def test_alignment_segments_and_counts(mrl, B, S_src, S_tgt, one_word):
    """Rows of several segments of 8192 positions, rows of up to and above the 256 positions that a block takes one per
    thread, words of 1, 63, 64 and more target tokens, fixed-point rounding of values over the whole range."""
    from oracle import thl_oracle
    from workloads import synth
    b = synth.make_thl(B, S_src, S_tgt, seed=S_tgt)
    if one_word:
        cut = [1, 63, 64, 65, 640]                     # tokens of word 0 in row i, the rest are word 1
        n = b["tgt_word_map"].shape[1]
        for i in range(B):
            b["src_word_map"][i] = torch.arange(S_src, device="cuda", dtype=torch.int32) % 2
            b["tgt_word_map"][i] = (torch.arange(n, device="cuda") >= cut[i % 5]).int()
        b["max_words"] = 2
    g = torch.Generator("cuda").manual_seed(1)
    b["src_logp"] = -torch.exp(12 * torch.randn(b["src_logp"].shape, device="cuda", generator=g)).clamp(max=2.0 ** 22)      # a word sums up to 257 of them: below 2^31
    out, bad = mrl.thl_word_align(b["src_logp"], b["src_mask"], b["src_word_map"], b["src_map_len"], b["tgt_mask"],
                                  b["tgt_word_map"], b["tgt_map_len"], b["max_words"])
    torch.cuda.synchronize()
    c = {k: (v.cpu().numpy() if isinstance(v, torch.Tensor) else v) for k, v in b.items()}
    want = thl_oracle.word_align_logprobs(c["src_logp"].astype(np.float64), c["src_mask"], c["src_word_map"], c["src_map_len"],
                                          c["tgt_mask"], c["tgt_word_map"], c["tgt_map_len"], -100.0)
    # a word's sum is exact to 2^-33 per source token, the output rounded to fp32
    assert np.all(np.abs(out.cpu().numpy() - want) <= 1e-6 + 2.0 ** -23 * np.abs(want))
    assert int(bad.item()) == 0


def test_alignment_of_a_row_that_ends_below_2_31(mrl):
    """The last segment of 8192 positions reaches beyond the largest 32-bit signed position; its tokens are found and
    nothing behind the row is read."""
    S = 2 ** 31 - 4096
    lp, mask = torch.zeros((1, S), device="cuda"), torch.zeros((1, S), dtype=torch.uint8, device="cuda")
    wmap = torch.zeros((1, S), dtype=torch.int32, device="cuda")
    at = [0, 300, 8192, S - 8191, S - 2, S - 1]
    for k, j in enumerate(at):
        lp[0, j] = -2.0 ** k
        mask[0, j] = 1
        wmap[0, k] = k // 2
    t = lambda v, dt: torch.tensor(v, dtype=dt, device="cuda")
    out, bad = mrl.thl_word_align(lp, mask, wmap, t([6], torch.int32), t([[1] * 4], torch.uint8), t([[0, 1, 2, 2]], torch.int32),
                                  t([4], torch.int32), 3)
    # sums of powers of two and halves of them are exact
    assert out.cpu().tolist() == [[-3.0, -12.0, -24.0, -24.0]]
    assert int(bad.item()) == 0


@pytest.mark.parametrize("B,T,G,agg", [(300, 3, 4, 0), (2049, 2, 700, 1), (4500, 1, 4096, 0), (9001, 2, 4097, 0), (20000, 1, 20000, 0),
                                       (3, 1024, 2, 0), (3, 1025, 2, 0), (2, 16384, 1, 0), (40, 1024, 4, 1), (33, 1030, 4, 0), (2, 20001, 1, 0)])
def test_sequence_weights_of_many_groups(mrl, B, T, G, agg):
    """Group counts up to and above the 4096 that fit LDS, steps of sequences that end inside one, empty sequences, auxiliary
    rows, group ids outside [0, G); sequences counted by a wave (up to 1024 slots) and by a block, in the launch of up to
    32768 slots and in the one above."""
    d, V = 16, 40
    g = torch.Generator("cuda").manual_seed(B)
    N = B * T
    H, W = torch.randn((N, d), device="cuda", generator=g), 0.3 * torch.randn((V, d), device="cuda", generator=g)
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    mask = (torch.rand(N, device="cuda", generator=g) < 0.7).to(torch.uint8)
    gid = torch.randint(-1, G + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
    kind = (torch.rand(B, device="cuda", generator=g) < 0.1).to(torch.uint8)
    gid[0], kind[0], mask[0] = 0, 0, 1                   # one sequence at least has a weight
    adv = torch.randn(B, device="cuda", generator=g)
    z = H.double() @ W.double().t()
    lp = z.gather(1, y.long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    behav = (lp + 0.1 * (torch.rand(N, device="cuda", generator=g) - 0.5)).float()       # ratios inside the clip range
    cfg = mrl.LossConfig(kl_beta=0.0, sgt_lambda=0.1, loss_agg=agg, dh_dtype=mrl.F32)
    out = mrl.grpo_loss_fwd_bwd(H, W, y, mask, behav, None, adv, gid, kind, B, T, G, cfg)
    st = mrl.read_stats(out["stats"])
    L = mask.view(B, T).sum(1).double()
    ok = (gid >= 0) & (gid < G)
    grpo, aux = (kind == 0) & ok, (kind != 0) & (L > 0)
    count = torch.bincount(gid[grpo].long(), minlength=G)
    if agg:
        c = grpo / L[grpo].sum()
    else:
        c = torch.where(grpo, 1.0 / ((count > 0).sum() * count[gid.clamp(0, G - 1).long()].clamp(min=1) * L.clamp(min=1)), 0.0)
    c = torch.where(aux, 1.0 / (aux.sum() * L.clamp(min=1)), torch.where(grpo, c, 0.0)).double().repeat_interleave(T) * mask
    k, w = kind.repeat_interleave(T) != 0, torch.exp(lp - behav.double())
    A = adv.double().repeat_interleave(T)
    pg, sgt = -(c * w * A)[~k].sum(), -(c * lp)[k].sum()
    gr = torch.where(k, -0.1 * c, -c * w * A)
    dz = -gr[:, None] * torch.softmax(z, 1)
    dz[torch.arange(N, device="cuda"), y.long()] += gr
    # fp32 sums of at most 40 terms per row, fp64 sums over the rows
    assert abs(st["loss_pg"] - float(pg)) <= 2e-6 * float((c * w * A.abs()).sum()) and abs(st["loss_sgt"] - float(sgt)) <= 2e-6 * abs(float(sgt))
    want = dz @ W.double()
    error, size = float((out["dH"].double() - want).norm()), float(want.norm())
    assert 0 < size and error <= 1e-5 * size
    assert st["n_scored_tokens"] == int(mask.sum())


def test_alignment_of_values_outside_the_range(mrl):
    """Log-probs of 2^31 and more in magnitude and infinities saturate the 64-bit fixed point, NaN counts as 0; the other
    words of the row and the other rows are what they are without them."""
    odd = [-float("inf"), float("inf"), float("nan"), -1e20, 1e20, -2.0 ** 31, -3e38, 2.0 ** 31]
    n = len(odd)
    lp = torch.full((2, n + 2), -0.75, device="cuda")
    lp[0, 1:n + 1] = torch.tensor(odd, device="cuda")
    ones, ids = torch.ones((2, n + 2), dtype=torch.uint8, device="cuda"), torch.arange(n + 2, dtype=torch.int32, device="cuda").repeat(2, 1)
    length = torch.full((2,), n + 2, dtype=torch.int32, device="cuda")
    out, bad = mrl.thl_word_align(lp, ones, ids, length, ones, ids, length, n + 2)
    big = 2.0 ** 31
    assert out.cpu().tolist() == [[-0.75, -big, big, 0.0, -big, big, -big, -big, big, -0.75], [-0.75] * (n + 2)]
    assert int(bad.item()) == 0


def _both_paths(monkeypatch, call):
    """What `call` returns or raises through the binding's native part and without it."""
    from paper_2605_07244_amd import binding
    got = []
    for native in (True, False):
        monkeypatch.setattr(binding, "_native", native)
        try:
            r = call()
            torch.cuda.synchronize()
            got.append(tuple(r))
        except Exception as e:
            got.append((type(e), str(e)))
    return got


def _same(a, b):
    if isinstance(a, torch.Tensor) and isinstance(b, torch.Tensor):
        return a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b)
    return type(a) is type(b) and a == b


def test_native_binding_advantages(mrl, monkeypatch):
    g = torch.Generator("cuda").manual_seed(5)
    r = torch.rand(24, device="cuda", generator=g)
    gid = torch.arange(3, device="cuda").repeat_interleave(8).int()
    own = (torch.arange(24, device="cuda") % 2).to(torch.uint8)
    shift = torch.rand(3, device="cuda", generator=g)
    forms = [((r, gid, 3), {}), ((r.view(3, 8), gid, 3), dict(is_own=own, scored=own, in_stats=own, mode=2, mix_alpha=0.5, ddof=1)),
             ((r, gid, 3), dict(baseline_shift=shift, eps_norm=1)), ((torch.nn.Parameter(r), gid, 3), {}), ((r[:0], gid[:0], 3), {}),
             # refused: dtype, device, stride, sizes, options
             ((r.double(), gid, 3), {}), ((r.cpu(), gid, 3), {}), ((r, gid.long(), 3), {}), ((r[::2], gid[::2], 3), {}),
             ((r, gid, 3), dict(baseline_shift=shift[:2])), ((r, gid, 0), {}), ((r, gid, 3), dict(mode=7)), ((r, gid, 3), dict(ddof=5)),
             ((r, gid, 3), dict(is_own=own.float())), ((None, gid, 3), {}), ((r, None, 3), {})]
    for args, kw in forms:
        a, b = _both_paths(monkeypatch, lambda: mrl.group_advantages(*args, **kw))
        assert len(a) == len(b) and all(_same(p, q) for p, q in zip(a, b)), (kw, a, b)


def test_native_binding_outputs_without_memory(mrl):
    """A dispatch mode whose new tensors refuse their data pointer: an exception on either path, and the next call works."""
    from torch.utils._python_dispatch import TorchDispatchMode
    from workloads import synth

    class Locked(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            out = func(*args, **(kwargs or {}))
            torch._C._set_throw_on_mutable_data_ptr(out)
            return out

    r, gid = torch.rand(24, device="cuda"), torch.arange(3, device="cuda").repeat_interleave(8).int()
    t = synth.make_thl(6, 90, 120, seed=3)
    align = [t[k] for k in ("src_logp", "src_mask", "src_word_map", "src_map_len", "tgt_mask", "tgt_word_map", "tgt_map_len", "max_words")]
    for call in (lambda: mrl.group_advantages(r, gid, 3), lambda: mrl.thl_word_align(*align)):
        with Locked(), pytest.raises(RuntimeError, match="data pointer"):
            call()
        assert bool(torch.isfinite(call()[0]).all())


def test_native_binding_alignment(mrl, monkeypatch):
    from workloads import synth
    t = synth.make_thl(6, 90, 120, seed=3)
    args = [t[k] for k in ("src_logp", "src_mask", "src_word_map", "src_map_len", "tgt_mask", "tgt_word_map", "tgt_map_len")]
    forms = [(args, {}), (args, dict(ignore_value=-7.5, want_bad_count=False)), (args, dict(ignore_value=-3))]
    for i, bad in enumerate([args[0].double(), args[1].bool(), args[2].long(), args[3].cpu(), args[4][:, ::2], args[5][:, :5], None]):
        forms.append((args[:i] + [bad] + args[i + 1:], {}))
    for a7, kw in forms:
        if a7[5] is not None and a7[5].shape != args[5].shape:
            continue                                   # (sizes of the other arrays are not checked: not called)
        a, b = _both_paths(monkeypatch, lambda: mrl.thl_word_align(*a7, t["max_words"], **kw))
        assert len(a) == len(b) and all(_same(p, q) for p, q in zip(a, b)), (kw, a, b)
    for words in (0, 1 << 20):
        a, b = _both_paths(monkeypatch, lambda: mrl.thl_word_align(*args, words))
        assert len(a) == len(b) and all(_same(p, q) for p, q in zip(a, b)), (words, a, b)


@pytest.mark.parametrize("B,S_src,S_tgt", [(5, 768, 769), (3, 769, 40), (4, 1000, 1537), (3, 2048, 2048), (3, 30, 2048), (2, 2049, 2000)])
def test_alignment_with_kept_words(mrl, B, S_src, S_tgt):
    """Rows around the sizes whose target words stay in registers: against the oracle, bad word ids included."""
    from oracle import thl_oracle
    from workloads import synth
    t = synth.make_thl(B, S_src, S_tgt, seed=S_tgt)
    t["tgt_word_map"][0, :3] = t["max_words"]
    out, bad = mrl.thl_word_align(t["src_logp"], t["src_mask"], t["src_word_map"], t["src_map_len"], t["tgt_mask"], t["tgt_word_map"],
                                  t["tgt_map_len"], t["max_words"])
    torch.cuda.synchronize()
    c = {k: (v.cpu().numpy() if isinstance(v, torch.Tensor) else v) for k, v in t.items()}
    maps = np.where(c["tgt_word_map"] >= t["max_words"], -1, c["tgt_word_map"])
    want = thl_oracle.word_align_logprobs(c["src_logp"].astype(np.float64), c["src_mask"], c["src_word_map"], c["src_map_len"],
                                          c["tgt_mask"], maps, c["tgt_map_len"], -100.0)
    # fp32 output of sums exact to 2^-33 per term
    assert np.all(np.abs(out.cpu().numpy() - want) <= 1e-6 * np.maximum(1, np.abs(want)))
    used = (c["tgt_word_map"][0, :3] >= t["max_words"]) & (np.arange(3) < min(int(c["tgt_mask"][0].sum()), int(c["tgt_map_len"][0])))
    assert int(bad) == int(used.sum())
