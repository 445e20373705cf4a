"""Wait states the compiler does not see: its hazard pass leaves inline assembly alone, and the direct loads and the matrix products of the
GEMM kernels are written that way.  On gfx950 five wait states have to lie between a vector instruction that writes a scalar
register (v_readfirstlane of a buffer descriptor) and a vector-memory instruction that reads it; with fewer it may see the old value.
And a 16x16x32 product (four passes) has to be eight wait states old before anything but another product reads what it writes."""
import os
import re
import subprocess

import pytest

from paper_2605_07244_amd import build

LLVM = "/opt/rocm/llvm/bin"
NEEDED = 5
PRODUCT_NEEDED = 8
VMEM = ("buffer_", "global_", "flat_", "scratch_")


def _scalars(text):
    out = set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out | {int(a) for a in re.findall(r"\bs(\d+)\b", text)}


def _written(op, operands):
    """Scalar registers that a vector instruction writes: all or the second of its destinations (carries of 64-bit sums)."""
    if not op.startswith("v_"):
        return set()
    two = re.match(r"v_(add_co|sub_co|subrev_co|addc_co|subb_co|subbrev_co|mad_u64_u32|mad_i64_i32|div_scale)", op)
    return _scalars(",".join(operands[:2 if two else 1]))


def _parse(listing):
    """[(operation, operands)] and, for each, the instructions that may come before it."""
    code, at = [], {}
    for line in listing.splitlines():
        m = re.match(r"\s+([a-z][a-z0-9_]*)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m:
            at[int(m[3], 16)] = len(code)
            code.append((m[1], [o.strip() for o in m[2].split(",")], int(m[3], 16)))
    before = [[] for _ in code]
    for i, (op, operands, addr) in enumerate(code):
        if i + 1 < len(code) and op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before[i + 1].append(i)
        if op == "s_branch" or op.startswith("s_cbranch"):
            offset = int(operands[0].split()[0])
            target = at.get(addr + 4 + 4 * (offset - 65536 if offset >= 32768 else offset))
            if target is not None:
                before[target].append(i)
    return [(op, operands) for op, operands, _ in code], before


def _early(code, before, i, wanted, needed, written):
    """Predecessors of instruction i, along every path of fewer than `needed` wait states, that write one of the wanted registers."""
    found, seen, todo = [], {}, [(b, 0) for b in before[i]]
    while todo:
        b, states = todo.pop()
        if seen.get(b, needed) <= states:
            continue
        seen[b] = states
        op, operands = code[b]
        if wanted & written(op, operands):
            found.append(" ".join([op, *operands]))
            continue
        states += int(operands[0]) + 1 if op == "s_nop" else 1
        if states < needed:
            todo += [(c, states) for c in before[b]]
    return found


def hazards(listing):
    """(instruction, predecessor) for every scalar register that a vector-memory instruction reads too early."""
    code, before = _parse(listing)
    return [(" ".join([op, *operands]), early) for i, (op, operands) in enumerate(code) if op.startswith(VMEM)
            for early in _early(code, before, i, _scalars(",".join(operands)), NEEDED, _written)]


def _vectors(text):
    out = set()
    for f, a, b in re.findall(r"\b([av])\[(\d+):(\d+)\]", text):
        out |= {(f, r) for r in range(int(a), int(b) + 1)}
    return out | {(f, int(r)) for f, r in re.findall(r"\b([av])(\d+)\b", text)}


def product_hazards(listing):
    """The same for registers that a matrix product writes and another kind of instruction names too early."""
    code, before = _parse(listing)
    products = [i for i, (op, _) in enumerate(code) if op.startswith("v_mfma")]
    near = {j for i in products for j in range(i + 1, min(i + 1 + PRODUCT_NEEDED, len(code)))}
    near |= {j for j, b in enumerate(before) if any(k != j - 1 for k in b)}          # (and where branches meet)
    near |= {j + n for j in list(near) for n in range(PRODUCT_NEEDED) if j + n < len(code)}
    written = lambda op, operands: _vectors(operands[0]) if op.startswith("v_mfma") else set()
    return [(" ".join([op, *operands]), early) for i in sorted(near) for op, operands in [code[i]]
            if not op.startswith(("v_mfma", "s_")) for early in _early(code, before, i, _vectors(",".join(operands)), PRODUCT_NEEDED, written)]


def test_the_search_finds_what_it_is_for():
    early = "\n".join(f"\t{t}    // {4 * k:012X}: 00000000" for k, t in enumerate(
        ["v_readfirstlane_b32 s6, v6", "s_add_u32 m0, s75, s36", "v_add_u32_e32 v6, s35, v1",
         "buffer_load_dwordx4 v6, s[4:7], 0 offen lds", "s_endpgm"]))
    assert len(hazards(early)) == 1
    assert hazards(early.replace("s_add_u32 m0, s75, s36", "s_nop 3")) == []
    soon = early.replace("s_add_u32 m0, s75, s36", "v_mfma_f32_16x16x32_bf16 a[4:7], v[0:3], v[4:7], a[4:7]").replace(
        "v_add_u32_e32 v6, s35, v1", "v_accvgpr_read_b32 v6, a5")
    assert len(product_hazards(soon)) == 1 and product_hazards(soon.replace("a5", "a8")) == []


def test_registers_are_not_read_early(tmp_path):
    """Every kernel of the library, as it was built."""
    if not os.path.exists(f"{LLVM}/llvm-objdump"):
        pytest.skip("no llvm-objdump")
    here = tmp_path / "libmrl.so"
    here.write_bytes(open(build.LIB, "rb").read())
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", str(here)], cwd=tmp_path, check=True, capture_output=True)
    objects = [p for p in tmp_path.iterdir() if p.name.endswith("gfx950")]
    assert len(objects) == len(build.SOURCES)
    loads = 0
    for p in objects:
        listing = subprocess.run([f"{LLVM}/llvm-objdump", "-d", str(p)], check=True, capture_output=True, text=True).stdout
        assert hazards(listing) == [], p.name
        assert product_hazards(listing) == [], p.name
        loads += listing.count(" lds ")
    assert loads > 100                                  # (the direct loads of the GEMM kernels were among them)
