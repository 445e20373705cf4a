"""Wait states the compiler does not see: its hazard pass leaves inline assembly alone, and the direct loads of the GEMM kernels
are written that way.  On gfx950 five wait states have to lie between a vector instruction that writes a scalar
register (v_readfirstlane of a buffer descriptor) and a vector-memory instruction that reads it; with fewer it may see the old value."""
import os
import re
import subprocess

import pytest

from paper_2605_07244_amd import build

LLVM = "/opt/rocm/llvm/bin"
NEEDED = 5
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


def hazards(listing):
    """(instruction, its predecessor) for every scalar register that is read too early, along every path of up to five instructions."""
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
    found = []
    for i, (op, operands, _) in enumerate(code):
        if not op.startswith(VMEM):
            continue
        todo = [(b, 0, frozenset(_scalars(",".join(operands)))) for b in before[i]]
        while todo:
            b, states, wanted = todo.pop()
            bop, bops, _ = code[b]
            late = wanted & _written(bop, bops)
            if late:
                found.append((" ".join([op, *operands]), " ".join([bop, *bops])))
                continue
            states += int(bops[0]) + 1 if bop == "s_nop" else 1
            if states < NEEDED:
                todo += [(c, states, wanted) for c in before[b]]
    return found


def test_the_search_finds_what_it_is_for():
    early = "\n".join(f"\t{t}    // {4 * k:012X}: 00000000" for k, t in enumerate(
        ["v_readfirstlane_b32 s6, v6", "s_add_u32 m0, s75, s36", "v_add_u32_e32 v6, s35, v1",
         "buffer_load_dwordx4 v6, s[4:7], 0 offen lds", "s_endpgm"]))
    assert len(hazards(early)) == 1
    assert hazards(early.replace("s_add_u32 m0, s75, s36", "s_nop 3")) == []


def test_scalar_registers_are_not_read_early_by_vector_memory_instructions(tmp_path):
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
        loads += listing.count(" lds ")
    assert loads > 100                                  # (the direct loads of the GEMM kernels were among them)
