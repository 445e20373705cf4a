"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
symbol declared in include/*.h, and rejects bad arguments before touching a device."""
import ctypes
import os
import re
import struct
import subprocess
import time

import numpy as np
import pytest

import paper_2605_07244_amd as m
from paper_2605_07244_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    inc = os.path.join(ROOT, "include")
    text = "".join(open(os.path.join(inc, f)).read() for f in sorted(os.listdir(inc)) if f.endswith(".h"))
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mrl_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = m.lib()
    names = _declared_symbols()
    assert {"mrl_token_logprobs", "mrl_group_advantages", "mrl_grpo_loss_fwd_bwd"} <= set(names)
    for name in names:
        assert hasattr(lib, name), name


def test_version_and_status_strings():
    assert m.version() >= 100
    assert m.status_string(0) == "ok"
    for code in range(-9, 0):
        assert m.status_string(code) not in ("ok", "unknown status")
    assert m.status_string(-99) == "unknown status"


def test_stats_struct_size_matches_header():
    # 7 doubles + 6 int64 (see mrl_loss_stats)
    assert binding.STATS_BYTES == 104 and len(binding.STATS_FIELDS) == 13


P = ctypes.c_void_p
FAKE = P(0x1000)   # never dereferenced: validation fails first


def _cfg(**kw):
    return binding.LossConfig(**kw).to_c()


def test_token_logprobs_argument_errors():
    lib = m.lib()
    f = lib.mrl_token_logprobs
    assert f(None, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, FAKE, 1 << 20, None) == -1
    assert f(FAKE, FAKE, FAKE, None, 8, 128, 32, 1, None, None, FAKE, 1 << 20, None) == -1
    assert f(FAKE, FAKE, FAKE, None, 8, 64, 32, 7, FAKE, None, FAKE, 1 << 20, None) == -3
    assert f(FAKE, FAKE, FAKE, None, -1, 128, 32, 1, FAKE, None, FAKE, 1 << 20, None) == -2
    assert f(FAKE, FAKE, FAKE, None, 8, 0, 32, 1, FAKE, None, FAKE, 1 << 20, None) == -2
    assert f(FAKE, FAKE, FAKE, None, 8, 64, 0, 1, FAKE, None, FAKE, 1 << 20, None) == -2
    assert f(FAKE, FAKE, FAKE, None, 8, 36, 32, 1, FAKE, None, FAKE, 1 << 20, None) == -2   # bf16: d % 8
    assert f(FAKE, FAKE, FAKE, None, 0, 128, 32, 1, FAKE, None, None, 0, None) == 0          # N = 0: no-op
    assert f(FAKE, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, None, 0, None) == -6
    assert f(FAKE, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, P(0x1001), 1 << 20, None) == -6  # misaligned
    assert f(FAKE, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, FAKE, 16, None) == -6           # too small


def test_workspace_queries():
    assert m.token_logprobs_workspace(1024, 128, 1000, m.BF16) > 0
    assert m.token_logprobs_workspace(1024, 100, 1000, m.BF16) == 0      # invalid shape -> 0
    small = m.grpo_loss_workspace(4, 64, 128, 1000, m.BF16, m.LossConfig(chunk_rows=256))
    big = m.grpo_loss_workspace(4, 64, 128, 1000, m.BF16, m.LossConfig(chunk_rows=1024))
    assert 0 < small < big
    assert m.grpo_loss_workspace(4, 64, 128, 1000, m.BF16, m.LossConfig(chunk_rows=100)) == 0
    # the stress configuration fits comfortably into one GPU's HBM
    ws5 = m.grpo_loss_workspace(1024, 2048, 4096, 151936, m.BF16, m.LossConfig())
    assert 5e9 < ws5 < 40e9


def test_group_advantages_argument_errors():
    f = m.lib().mrl_group_advantages
    ok_tail = (FAKE, None, None, None, None)
    assert f(None, FAKE, None, None, None, None, 8, 2, 1, 1e-6, 0, 1.0, 0.2, 0.8, *ok_tail) == -1
    assert f(FAKE, FAKE, None, None, None, None, 8, 2, 1, 1e-6, 0, 1.0, 0.2, 0.8, None, None, None, None, None) == -1
    assert f(FAKE, FAKE, None, None, None, None, 8, 0, 1, 1e-6, 0, 1.0, 0.2, 0.8, *ok_tail) == -2
    assert f(FAKE, FAKE, None, None, None, None, -1, 2, 1, 1e-6, 0, 1.0, 0.2, 0.8, *ok_tail) == -2
    assert f(FAKE, FAKE, None, None, None, None, 8, 2, 5, 1e-6, 0, 1.0, 0.2, 0.8, *ok_tail) == -7
    assert f(FAKE, FAKE, None, None, None, None, 8, 2, 1, -1.0, 0, 1.0, 0.2, 0.8, *ok_tail) == -7
    assert f(FAKE, FAKE, None, None, None, None, 8, 2, 1, 1e-6, 2, 1.0, 0.2, 0.8, *ok_tail) == -7
    assert f(FAKE, FAKE, None, None, None, None, 8, 2, 1, 1e-6, 0, 1.5, 0.2, 0.8, *ok_tail) == -7
    assert f(FAKE, FAKE, None, None, None, None, 0, 2, 1, 1e-6, 0, 1.0, 0.2, 0.8, *ok_tail) == 0


def _loss(cfg, *, hidden=FAKE, ref=FAKE, B=4, T=8, G=2, d=128, V=100, dt=1, ws=FAKE, ws_bytes=1 << 30,
          stats=FAKE, seq_adv=FAKE):
    f = m.lib().mrl_grpo_loss_fwd_bwd
    return f(hidden, FAKE, FAKE, FAKE, FAKE, ref, seq_adv, FAKE, None, B, T, G, d, V, dt,
             ctypes.byref(cfg) if cfg is not None else None, FAKE, FAKE, FAKE, stats, ws, ws_bytes, None)


def test_loss_argument_errors():
    good = _cfg()
    assert _loss(good, hidden=None) == -1
    assert _loss(good, stats=None) == -1
    assert _loss(None) == -1
    assert _loss(good, ref=None) == -1                       # beta > 0 needs a reference trace
    assert _loss(good, B=0) == -2
    assert _loss(good, T=0) == -2
    assert _loss(good, G=0) == -2
    assert _loss(good, G=9) == -2                            # more groups than sequences
    assert _loss(good, d=65) == -2
    assert _loss(good, dt=3) == -3
    assert _loss(_cfg(clip_eps_low=-0.1)) == -7
    assert _loss(_cfg(kl_beta=-1.0)) == -7
    assert _loss(_cfg(loss_agg=2)) == -7
    assert _loss(_cfg(ratio_level=3)) == -7
    assert _loss(_cfg(ratio_level=1, loss_agg=1)) == -7
    assert _loss(_cfg(accumulate_dw=3)) == -7
    assert _loss(_cfg(dh_dtype=5)) == -7
    assert _loss(_cfg(chunk_rows=300)) == -7
    assert _loss(_cfg(scored_rows_hint=-5)) == -7
    assert _loss(_cfg(dh_dtype=1), dt=0) == -7               # fp32 path writes fp32 dH only
    assert _loss(good, ws=None) == -6
    assert _loss(good, ws_bytes=1024) == -6


def test_no_device_is_an_error_not_a_fallback():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is visible")
    # all arguments valid: the call must stop at the device check, nothing is computed on the CPU
    rc = _loss(_cfg())
    assert rc in (-8, -9)


def test_profile_calls_without_device():
    assert m.lib().mrl_profile_enable(0) == 0
    assert m.lib().mrl_profile_collect(None, None) == -1
    out = m.profile_collect()
    assert set(out) == set(m.PROF_CLASSES)


def test_probe_argument_errors():
    f = m.lib().mrl_probe_mfma_rate
    out = ctypes.c_double(0.0)
    assert f(0, 0.1, None, 1 << 20, ctypes.byref(out)) == -1
    assert f(0, 0.1, FAKE, 1 << 20, None) == -1
    assert f(0, 0.0, FAKE, 1 << 20, ctypes.byref(out)) == -7
    assert f(0, 60.0, FAKE, 1 << 20, ctypes.byref(out)) == -7


def test_dw_tail_plan_host_logic():
    """The plan of the dW launch's K-split tail: every item of every split tile is dealt to exactly one XCD,
    the partial-tile scratch (256 tiles) is never exceeded, whole super-tile rows are left alone."""
    f = m.lib().mrl_diag_dw_tail_plan
    out = (ctypes.c_int32 * 12)()
    assert f(1000, 64, None) == -1 and f(0, 64, out) == -2 and f(1000, 0, out) == -2
    seen_split = set()
    for V in (300, 2048, 2500, 3001, 8333, 32000, 50257, 128256, 151936, 262144):
        for d in (64, 384, 768, 1536, 2048, 3584, 4096, 5120, 8192):
            assert f(V, d, out) == 0
            m0, rows, split = out[0], out[1], out[2]
            pre = list(out[3:12])
            Mt, Nt = -(-V // 256), -(-d // 256)
            sup_m = 16 if Nt == 1 else 8
            assert m0 % sup_m == 0 and m0 + rows == Mt and 0 <= rows < sup_m
            assert split == 0 or 2 <= split <= 8
            if split:
                items = rows * Nt * split
                assert m0 > 0 and rows > 0 and items <= 256
                assert pre[0] == 0 and pre[8] == items and all(a <= b for a, b in zip(pre, pre[1:]))
            else:
                assert pre == [0] * 9
            seen_split.add(split)
    assert 0 in seen_split and 8 in seen_split and len(seen_split) >= 3
    # the benchmark shapes: V = 151936 leaves two ragged tile rows
    assert f(151936, 4096, out) == 0 and (out[0], out[1], out[2]) == (592, 2, 8) and list(out[3:12]) == list(range(0, 257, 32))
    assert f(151936, 1536, out) == 0 and out[2] >= 2 and out[11] == 12 * out[2]


def _modelled_tail_plan(V, d):
    """The dW tail plan from its definition: every compute unit by itself, each item on the one that is free first."""
    Mt, Nt = -(-V // 256), -(-d // 256)
    sup_m, sup_n = (8, 4) if Nt % 4 == 0 else (16, 1) if Nt == 1 else (8, 2)
    rows = Mt % sup_m
    m0, tiles, cols = Mt - rows, rows * Nt, -(-Nt // sup_n)
    plan = [m0, rows, 0] + [0] * 9
    if tiles == 0 or m0 == 0:
        return plan

    def per_xcd(rows_m):
        t = [0] * 8
        for s in range(-(-rows_m // sup_m) * cols):
            t[s % 8] += min(sup_m, rows_m - s // cols * sup_m) * min(sup_n, Nt - s % cols * sup_n)
        return t

    best = max(-(-t // 32) for t in per_xcd(Mt)) - 0.02
    whole = per_xcd(m0)
    for split in range(2, 9):
        if tiles * split > 256:
            break
        free = np.array([[t // 32 + (c < t % 32) for c in range(32)] for t in whole], dtype=np.float64)
        end, count = free.max(), [0] * 8
        for _ in range(tiles * split):
            x, c = divmod(int(free.argmin()), 32)
            free[x, c] += 1.0 / split + 0.02
            end = max(end, free[x, c])
            count[x] += 1
        if end < best - 1e-9:
            best = end
            plan[2:] = [split] + [sum(count[:x]) for x in range(9)]
    return plan


def test_dw_tail_plan_is_the_modelled_one_and_cheap():
    f = m.lib().mrl_diag_dw_tail_plan
    out = (ctypes.c_int32 * 12)()
    for V in (2100, 4099, 8333, 32000, 50257, 128256, 151936):
        for d in (64, 512, 712, 1536, 2048, 3584, 4096):
            assert f(V, d, out) == 0 and list(out) == _modelled_tail_plan(V, d), (V, d)
    # it runs on the host in every dW launch, the shortest of which take some 100 us: a few microseconds, and
    # here at most a twentieth of what one unit after the other took
    took = []
    for _ in range(20):
        t = time.perf_counter()
        f(151936, 4096, out)
        took.append(time.perf_counter() - t)
    assert min(took) < 35e-6


def test_dh_split_is_the_earliest_end():
    """Slices of the dH launch's last round: the smallest count whose rounds of 256 items end earliest (an item costs its share
    and a fiftieth of a tile), no slice below 16 panels, no more items than the scratch holds."""
    from fractions import Fraction
    f = m.lib().mrl_diag_dh_split
    assert f(0, 100, 256) == -2 and f(256, 100, 256) == -2 and f(1, 0, 256) == -2 and f(10, 100, 9) == -2
    for tiles in list(range(1, 34)) + [64, 85, 86, 120, 127, 128, 129, 200, 254, 255]:
        for panels in (2, 16, 31, 32, 48, 160, 782, 1023, 1024, 2374, 4096):
            for room in (256, 300, 512, 777, 1024):
                best, end = 1, Fraction(1)
                for s in range(2, min(64, panels // 16, room // tiles) + 1):
                    e = -(-tiles * s // 256) * (Fraction(1, s) + Fraction(1, 50))
                    if e < end:
                        best, end = s, e
                assert f(tiles, panels, room) == best, (tiles, panels, room)


def _cut_cases():
    for V in (300, 1000, 2048, 8192, 32000, 50257, 128256, 151936):
        for d in (64, 512, 712, 1024, 1536, 4096, 8192):
            for chunk in (512, 1024, 2560, 5120, 16384, 65536):
                for rows in sorted({1, 128, 129, 256, 257, 384, 385, 640, 1000, 1877, 2000, 3000, 5000, 16384, 16385, chunk - 1, chunk}):
                    if rows <= chunk:
                        yield V, d, chunk, rows


def test_tiles_of_the_large_launches_cover_their_rows():
    """For every count of valid rows: the tiles cover the rows, the workgroups launched are as many as the device deals out (whole
    rounds of 256, then the last round's slices, to 8 XCDs), and the slices fit the scratch."""
    f, out = m.lib().mrl_diag_gemm_cut, (ctypes.c_int32 * 9)()
    assert f(2, 1, 1, 256, 1000, 64, 0, None) == -1
    for bad in ((3, 1, 1, 256, 1000, 64, 0), (2, 0, 1, 256, 1000, 64, 0), (2, 257, 1, 256, 1000, 64, 0), (2, 1, 1, 200, 1000, 64, 0),
                (5, 1, 1, 256, 0, 64, 0), (5, 1, 1, 256, 1000, 60, 0), (6, 1, 0, 256, 1000, 64, 0), (6, 1, 1, 256, 1000, 64, -1)):
        assert f(*bad, out) == -2, bad
    dealt = lambda whole, items: whole + -(-items // 8) * 8
    cuts = {m.GEMM_FWD: set(), m.GEMM_DH: set()}
    for V, d, chunk, rows in _cut_cases():
        for launch, other in ((m.GEMM_FWD, -(-V // 256)), (m.GEMM_DH, -(-d // 256))):
            if launch == m.GEMM_FWD and chunk > 16384:
                continue
            for room in (0, 300) if launch == m.GEMM_DH else (0,):
                c = m.gemm_cut(launch, rows, V, d, chunk, 0, room)
                at = (launch, V, d, chunk, rows, room, c)
                long = 384 * c["wide"] + 256 * c["narrow"] + 128 * c["half"]
                last = 128 if c["half"] else 256 if c["narrow"] else 384
                assert c["last_start"] < rows <= long and c["last_start"] == long - last, at
                assert c["tiles"] == (c["wide"] + c["narrow"] + c["half"]) * other and c["rest"] == c["tiles"] % 256, at
                assert c["split"] == 1 or c["rest"] * c["split"] <= c["tail_items"], at
                assert dealt(c["tiles"] - c["rest"], c["rest"] * c["split"]) <= c["blocks"], at
                if launch == m.GEMM_DH:
                    assert c["half"] == 0 or (c["wide"] + c["narrow"] == 0 and c["tiles"] <= 256), at
                cuts[launch].add((c["wide"] > 0, c["narrow"] > 0, c["half"] > 0))
        for room in (0, 171):
            c = m.gemm_cut(m.GEMM_DW, rows, V, d, chunk, chunk, room)
            if c["wide"]:
                assert c["tiles"] == -(-V // 384) * -(-d // 256) and c["rest"] == c["tiles"] % 256
                assert c["split"] == 1 or c["rest"] * c["split"] <= c["tail_items"]
                assert dealt(c["tiles"] - c["rest"], c["rest"] * c["split"]) <= c["blocks"]
    assert len(cuts[m.GEMM_FWD]) >= 5 and len(cuts[m.GEMM_DH]) >= 4


@pytest.mark.parametrize("rows,d,V,cut", [
    (5814, 1536, 21132, (0, 23, 0)), (8874, 792, 5427, (0, 35, 0)),     # 16 or 24 columns of 384 and 256: the shorter ones would lie on the same XCDs in every band
    (2814, 744, 151936, (6, 2, 0)), (3000, 1536, 151936, (8, 0, 0)),
])
def test_forward_columns_of_two_kinds(rows, d, V, cut):
    c = m.gemm_cut(m.GEMM_FWD, rows, V, d, 15360)
    assert (c["wide"], c["narrow"], c["half"]) == cut


def test_a_pass_holds_up_to_65536_rows():
    """A call of up to 65536 slots is one pass: its stash grows with every 256 slots up to there, and not beyond."""
    f = m.lib().mrl_grpo_loss_workspace
    size = lambda N: f(1, N, 64, 1000, 1, None)
    stash = 256 * (1024 + 64) * 2
    for N in (61440, 65280):
        assert size(N + 256) - size(N) >= stash, N
    assert size(65536 + 256) - size(65536) < stash


def test_thl_word_align_argument_errors():
    f = m.lib().mrl_thl_word_align
    args = lambda **kw: [kw.get("p0", FAKE), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, kw.get("B", 4), kw.get("S", 16), 16,
                         kw.get("W", 32), ctypes.c_float(-100.0), kw.get("out", FAKE), None, None]
    assert f(*args(p0=None)) == -1
    assert f(*args(out=None)) == -1
    assert f(*args(S=0)) == -2
    assert f(*args(B=-1)) == -2
    assert f(*args(W=0)) == -2
    assert f(*args(W=8193)) == -2
    assert f(*args(B=0)) == 0          # empty batch: no-op


def test_token_scores_argument_errors():
    lib = m.lib()
    f = lib.mrl_token_scores
    assert f(None, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, None, FAKE, 1 << 20, None) == -1
    assert f(FAKE, FAKE, FAKE, None, 8, 36, 32, 1, FAKE, None, FAKE, FAKE, 1 << 20, None) == -2
    assert f(FAKE, FAKE, FAKE, None, 8, 128, 32, 1, FAKE, None, FAKE, FAKE, 16, None) == -6    # workspace too small
    assert f(FAKE, FAKE, FAKE, None, 0, 128, 32, 1, FAKE, None, FAKE, None, 0, None) == 0
    # the entropy needs a third partial buffer: its workspace is the larger one
    assert lib.mrl_token_scores_workspace(4096, 256, 4000, 1) > lib.mrl_token_logprobs_workspace(4096, 256, 4000, 1)


def test_static_logprobs_argument_errors():
    """The allocation-free variant validates on the host before it touches a device: NULL
    pointers, shapes, and inputs beyond its built-in scratch buffer."""
    f = m.lib().mrl_token_logprobs_static
    one = 8  # any non-null address: rejected arguments are never dereferenced
    assert f(None, one, one, None, 16, 128, 512, 1, one, None, None) == -1
    assert f(one, one, one, None, 16, 100, 512, 1, one, None, None) == -2        # d % 8
    assert f(one, one, one, None, 16, 128, 512, 7, one, None, None) == -3
    assert f(one, one, one, None, 0, 128, 512, 1, one, None, None) == 0           # empty input: no-op
    assert f(one, one, one, None, 1 << 23, 128, 512, 1, one, None, None) == -10   # 8 B per row > 32 MiB
    assert f(one, one, one, None, 1024, 128, 1 << 22, 1, one, None, None) == -10  # partials of one pass > 32 MiB
    assert "scratch" in m.status_string(-10)


def _kernel_notes(tmp_path):
    """The kernel descriptions (name -> {property: value}) of every gfx950 code object in the built library."""
    blob = open(os.path.join(ROOT, "paper_2605_07244_amd", "libmrl.so"), "rb").read()
    kernels = {}
    for at in (x.start() for x in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob)):
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" not in name or size == 0:
                continue
            path = tmp_path / "code_object"
            path.write_bytes(blob[at + offset:at + offset + size])
            text = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n  - ", text)[1:]:
                props = dict(re.findall(r"^\s*\.(\w+):\s+(\S+)$", part, flags=re.M))
                if "private_segment_fixed_size" in props:
                    kernels[re.findall(r"^    \.name:\s+(\S+)$", part, flags=re.M)[0]] = props
    return kernels


def test_no_kernel_uses_scratch_memory(tmp_path):
    """Spills and address-selected locals: their reloads wait for every vector-memory access issued before them.
    (k_mfma_rate, the probe of the matrix cores' rate, is no part of any call.)"""
    kernels = {k: p for k, p in _kernel_notes(tmp_path).items() if "k_mfma_rate" not in k}
    assert len(kernels) >= 25 and sum("gemm_nt_bf16" in k for k in kernels) == 3
    assert {k: p["private_segment_fixed_size"] for k, p in kernels.items() if p["private_segment_fixed_size"] != "0"} == {}


def test_native_binding_is_optional(tmp_path, monkeypatch):
    """The CPython extension only marshals faster: where it is missing, broken or built against another torch, the binding
    warns once and every call goes through ctypes; so does a build that cannot compile it."""
    import shutil

    m.lib()                                                      # (the C library itself is not optional)
    here = binding._HERE
    host = os.path.join(here, "mrl_host.so")
    assert os.path.exists(host) and binding._load_host().torch_version == binding.torch.__version__
    monkeypatch.setattr(binding, "_HERE", str(tmp_path))
    for content in (None, b"", b"not a shared object"):
        if content is not None:
            (tmp_path / "mrl_host.so").write_bytes(content)
        monkeypatch.setattr(binding, "_HOST", None)
        with pytest.warns(RuntimeWarning, match="ctypes"):
            none = binding._host()
        assert none.advantages(*range(14)) is None and none.align(*range(11)) is None
        assert binding._host() is none                           # (once)
    monkeypatch.setattr(binding, "_HERE", here)
    monkeypatch.setattr(binding, "_HOST", None)
    monkeypatch.setattr(binding.torch, "__version__", "0.0")
    with pytest.warns(RuntimeWarning, match="built against torch"):
        assert binding._host().advantages(*range(14)) is None

    from paper_2605_07244_amd import build
    shutil.copy(host, tmp_path / "mrl_host.so")
    monkeypatch.setattr(build, "HOST", str(tmp_path / "mrl_host.so"))
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert build._build_host(False) is False and not (tmp_path / "mrl_host.so").exists()
