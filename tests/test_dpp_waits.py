"""A DPP instruction reads its first source from other lanes, and may do so no sooner than two wait states behind a vector
instruction that writes that register.  The compiler sees to that, but not for inline assembly, which the pivots of the
initialization's triangular factors are written in.  The check runs over the AMD assembly of the library as it was built here."""
import os
import subprocess

import pytest

import paper_2510_24061_amd as fq
from test_lds_waits import OBJDUMP, _code_objects, _functions, _registers

ADD = "v_fmac_f64_dpp"                                # written in inline assembly only
WAIT = 2


def _is_dpp(mnemonic, operands):
    return mnemonic.startswith("v_") and (mnemonic.endswith("_dpp") or "row_newbcast" in operands or "quad_perm" in operands)


def _states(mnemonic, operands):
    return int(operands.split()[0], 0) + 1 if mnemonic == "s_nop" else 1


def _faults(code):
    """(address, mnemonic, operands) of the DPP reads that follow a write of their source too closely, on any path"""
    index = {ins[0]: i for i, ins in enumerate(code)}
    before = {}
    for i, (_, mn, _, target) in enumerate(code):
        if target is not None:
            before.setdefault(index[target], []).append(i)
        if mn not in ("s_branch", "s_endpgm") and i + 1 < len(code):
            before.setdefault(i + 1, []).append(i)
    bad = []
    for i, (addr, mn, ops, _) in enumerate(code):
        if not _is_dpp(mn, ops):
            continue
        source = _registers(ops.split(",")[1])
        work = [(p, 0) for p in before.get(i, [])]
        while work:
            j, passed = work.pop()
            _, m, o, _ = code[j]
            if m.startswith("v_") and m != "v_nop" and _registers(",".join(o.split(",")[:2] if "swap" in m else o.split(",")[:1])) & source:
                bad.append((addr, mn, ops.strip()))
                break
            passed += _states(m, o)
            if passed < WAIT:
                work += [(p, passed) for p in before.get(j, [])]
    return bad


def _own_wait(code):
    """Inline additions with something else than a wait or another of them right before"""
    return [c[:3] for p, c in zip([(0, "", "", None)] + code, code)
            if c[1] == ADD and p[1] != ADD and not (p[1] == "s_nop" and _states(*p[1:3]) >= WAIT)]


def _code(*lines):
    return [(4 * i, *(ln.split(" ", 1) + [""])[:2], 4 * int(t) if t else None)
            for i, (ln, t) in enumerate(l if isinstance(l, tuple) else (l, None) for l in lines)]


def test_the_check_itself():
    add = "v_fmac_f64_dpp v[2:3], v[2:3], v[8:9] row_newbcast:1 row_mask:0xf bank_mask:0xf"
    copy, other = "v_mov_b32_e32 v3, v40", "v_mov_b32_e32 v4, v40"
    assert _faults(_code(copy, add, "s_endpgm")) and _faults(_code(copy, other, add, "s_endpgm"))
    assert _faults(_code(copy, "s_nop 0", add, "s_endpgm"))
    assert not _faults(_code(copy, "s_nop 1", add, "s_endpgm")) and not _faults(_code(copy, other, other, add, "s_endpgm"))
    # the write is at the end of a loop, the read at its head; a compiler's DPP move right behind the assembly
    assert _faults(_code(other, other, add, other, copy, ("s_cbranch_scc1 x", "2"), "s_endpgm"))
    assert _faults(_code("s_nop 1", add, "v_mov_b64_dpp v[6:7], v[2:3] row_newbcast:2 row_mask:0xf bank_mask:0xf", "s_endpgm"))
    assert _own_wait(_code(other, add, "s_endpgm")) and not _own_wait(_code("s_nop 1", add, add, "s_endpgm"))


def test_no_lane_is_read_too_early(tmp_path):
    if not os.path.exists(fq.lib_path()):
        pytest.skip("library not built")
    kernels, adds, faults = 0, 0, {}
    for i, obj in enumerate(_code_objects(fq.lib_path())):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout
        for name, code in _functions(text).items():
            if not any(_is_dpp(mn, ops) for _, mn, ops, _ in code):
                continue
            kernels += 1
            adds += any(mn == ADD for _, mn, _, _ in code)
            bad = _faults(code) + _own_wait(code)
            if bad:
                faults[name] = bad
    assert kernels >= 40 and adds == 14               # triangular factors: two forms for each of seven sizes
    assert not faults, "\n".join(f"{n}: {len(b)} instructions, first {b[:3]}" for n, b in faults.items())
