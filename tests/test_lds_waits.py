"""The transposing LDS reads of the product kernels are written as inline assembly, whose completion the
compiler does not track: nothing but the kernel's own waits keeps an instruction from touching a
destination register while its data is still on the way.  The check runs over the AMD assembly of the library as
it was built here: on no path through a kernel does any instruction read or write such a register before
a wait that covers the read."""
import os
import re
import struct
import subprocess

import pytest

import paper_2510_24061_amd as fq

OBJDUMP = os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
READ = "ds_read_b64_tr_b8"
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _code_objects(path):
    """gfx950 code objects in the bundles of a host library."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        count, p = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + off:at + off + size]
            p += 24 + length
        at = data.find(MAGIC, at + len(MAGIC))


def _registers(operands):
    return {(kind, i) for kind, one, lo, hi in REG.findall(operands)
            for i in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))}


def _functions(text):
    """name -> list of (address, mnemonic, operands, branch target or None)"""
    out, body = {}, None
    for line in text.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if head:
            body = out.setdefault(head.group(2), [])
            base = int(head.group(1), 16)
            continue
        m = re.match(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+):", line)
        if m and body is not None:
            target = None
            if m.group(1).startswith(("s_cbranch", "s_branch")):
                target = base + int(re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$", line).group(1) or "0", 16)
            body.append((int(m.group(3), 16), m.group(1), m.group(2), target))
    return out


def _step(pending, mnemonic, operands):
    """State after one instruction: register -> LDS operations issued behind the read that fills it.  Returns
    (state, registers touched while pending)."""
    if mnemonic == "s_waitcnt":
        m = re.search(r"lgkmcnt\((\d+)\)", operands)
        raw = re.match(r"\s*(0x[0-9a-f]+|\d+)\s*$", operands)
        left = int(m.group(1)) if m else (int(raw.group(1), 0) >> 8) & 15 if raw else 15
        # LDS operations complete in order: with at most `left` outstanding, a read followed by that many is done
        return ({r: n for r, n in pending.items() if n < left} if left < 15 else pending), ()
    touched = _registers(operands) & pending.keys() if pending else ()
    if mnemonic.startswith("ds_"):
        pending = {r: min(n + 1, 15) for r, n in pending.items()}
        if mnemonic == READ:
            pending.update((r, 0) for r in _registers(operands.split(",")[0]))
    return pending, touched


def _faults(code):
    """(address, mnemonic, operands) of the instructions that touch a destination too early"""
    index = {ins[0]: i for i, ins in enumerate(code)}
    starts = sorted({0} | {index[t] for *_, t in code if t is not None} |
                    {i + 1 for i, (_, mn, _, t) in enumerate(code) if t is not None or mn == "s_endpgm"})
    starts = [s for s in starts if s < len(code)]
    end = dict(zip(starts, starts[1:] + [len(code)]))
    entry, work, bad = {0: {}}, [0], set()
    while work:
        s = work.pop()
        state = dict(entry[s])
        for i in range(s, end[s]):
            addr, mn, ops, _ = code[i]
            assert not mn.startswith(("s_setpc", "s_swappc")), "calls are not followed"
            state, touched = _step(state, mn, ops)
            if touched:
                bad.add((addr, mn, ops.strip()))
        _, mn, _, target = code[end[s] - 1]
        nxt = [index[target]] if target is not None else []
        if mn not in ("s_branch", "s_endpgm") and end[s] < len(code):
            nxt.append(end[s])
        for t in nxt:
            old = entry.get(t)
            new = dict(state) if old is None else {**old, **{r: min(n, old.get(r, n)) for r, n in state.items()}}
            if new != old:
                entry[t] = new
                work.append(t)
    return sorted(bad)


def test_the_check_itself():
    """A copy before the wait, on a back edge, is found; the same copy behind the wait is not."""
    def code(*lines):
        return [(4 * i, *(ln.split(" ", 1) + [""])[:2], 4 * int(t) if t else None)
                for i, (ln, t) in enumerate(l if isinstance(l, tuple) else (l, None) for l in lines)]
    early = code("ds_read_b64_tr_b8 v[2:3], v9", ("s_cbranch_scc1 x", "3"), "s_endpgm", "v_mov_b32 v7, v3",
                 "s_waitcnt lgkmcnt(0)", ("s_branch x", "0"))
    late = code("ds_read_b64_tr_b8 v[2:3], v9", ("s_cbranch_scc1 x", "3"), "s_endpgm", "s_waitcnt lgkmcnt(0)",
                "v_mov_b32 v7, v3", ("s_branch x", "0"))
    counted = code("ds_read_b64_tr_b8 v[2:3], v9", "ds_read_b128 v[12:15], v9", "s_waitcnt vmcnt(3) lgkmcnt(1)",
                   "v_mov_b32 v7, v3", "s_endpgm")
    assert [f[0] for f in _faults(early)] == [12] and _faults(late) == [] and _faults(counted) == []


def test_no_register_is_touched_before_its_transposing_read_has_landed(tmp_path):
    if not os.path.exists(fq.lib_path()):
        pytest.skip("library not built")
    kernels, faults = 0, {}
    for i, obj in enumerate(_code_objects(fq.lib_path())):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout
        if READ not in text:
            continue
        for name, code in _functions(text).items():
            if any(mn == READ for _, mn, _, _ in code):
                kernels += 1
                bad = _faults(code)
                if bad:
                    faults[name] = bad
    assert kernels >= 12                           # every product with a [K, N] operand, and the adapter gradient's
    assert not faults, "\n".join(f"{n}: {len(b)} instructions, first {b[:3]}" for n, b in faults.items())
