"""The step-prefill kernel writes its matrix instructions as inline assembly, for which the
compiler keeps no wait states.  This reads the built device code and follows every path through
those kernels: no operand of a matrix instruction is written by a vector instruction less than
two issue slots before it, and nothing but an accumulation into the same registers touches a
result less than 18 slots after it (a matrix instruction is issued 8 slots after the one before
it at the earliest)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2502_13575_amd as ets

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
WRITE_TO_MATRIX, MATRIX_TO_USE, MATRIX_ISSUE = 2, 18, 8


def _disassembly(tmp_path):
    ets.load_library()
    lib = os.path.join(os.path.dirname(ets.__file__), "libetsattn.so")
    fat, obj = str(tmp_path / "fat.bin"), str(tmp_path / "dev.o")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "-O", "binary", "--only-section=.hip_fatbin",
                    lib, fat], check=True)
    data = open(fat, "rb").read()
    assert data.startswith(b"__CLANG_OFFLOAD_BUNDLE__")
    at = 32
    for _ in range(struct.unpack_from("<Q", data, 24)[0]):
        offset, size, n = struct.unpack_from("<QQQ", data, at)
        if b"gfx950" in data[at + 24:at + 24 + n]:
            open(obj, "wb").write(data[offset:offset + size])
        at += 24 + n
    return subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", obj],
                          check=True, capture_output=True, text=True).stdout


def _registers(operand):
    m = re.search(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", operand)
    if not m:
        return frozenset()
    first, last = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return frozenset((m[1], i) for i in range(first, last + 1))


def _functions(text):
    """{name: [(address, mnemonic, operands, branch target or None)]}"""
    out, name, start = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if m:
            name, start = m[2], int(m[1], 16)
            out[name] = []
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):[^<]*(?:<[^>]*\+0x([0-9a-f]+)>)?", line)
        if m and name:
            ops = re.split(r",\s*(?![^\[]*\])", m[2]) if m[2] else []
            out[name].append((int(m[3], 16), m[1], ops, start + int(m[4], 16) if m[4] else None))
    return out


def _step(state, mnemonic, ops):
    """State after an instruction and what it breaks.  state: {(kind, register): slots since it was
    written}, kind "w" by the vector unit or "m" by a matrix instruction; ("pipe",): slots since
    the last matrix instruction."""
    faults = []
    regs = [_registers(o) for o in ops]
    if mnemonic.startswith("v_mfma"):
        stall = max(0, MATRIX_ISSUE - state.get(("pipe",), MATRIX_ISSUE))
        state = {k: a + stall if k[0] == "m" else a for k, a in state.items()}
        for r in regs[1] | regs[2] | regs[3]:
            if state.get(("w", r), WRITE_TO_MATRIX) < WRITE_TO_MATRIX:
                faults.append("vector write of %s%d" % r)
        accumulates = regs[0] == regs[3]
        for r in regs[1] | regs[2] | (frozenset() if accumulates else regs[0] | regs[3]):
            if state.get(("m", r), MATRIX_TO_USE) < MATRIX_TO_USE:
                faults.append("matrix result %s%d" % r)
        if accumulates and any(("m", r) in state for r in regs[0]):
            whole = {state.get(("m", r)) for r in regs[0]}
            if len(whole) != 1:
                faults.append("part of a matrix result %s" % ops[0])
    else:
        for r in frozenset().union(*regs) if regs else ():
            if state.get(("m", r), MATRIX_TO_USE) < MATRIX_TO_USE:
                faults.append("matrix result %s%d" % r)
    slots = int(ops[0], 0) + 1 if mnemonic == "s_nop" else 1
    if mnemonic.startswith("v_mfma"):
        written = {("m", r): 0 for r in regs[0]}
        written[("pipe",)] = 0
    elif mnemonic.startswith("v_") and ops:
        both = frozenset().union(*regs) if "swap" in mnemonic else regs[0]
        written = {("w", r): 0 for r in both}
    else:
        written = {}
    limit = {"w": WRITE_TO_MATRIX, "m": MATRIX_TO_USE, "pipe": MATRIX_ISSUE}
    nxt = {k: a for k, a in state.items() if k not in written}
    for k in [k for k in nxt if len(k) > 1 and (("w" if k[0] == "m" else "m"), k[1]) in written]:
        del nxt[k]
    nxt.update(written)
    # an instruction's own writes are `slots - slots` old when the next one issues: age 0
    return {k: a + (slots if k not in written else 0) for k, a in nxt.items()
            if a + (slots if k not in written else 0) < limit[k[0]]}, faults


def _check(code):
    """Faults of one function over all its paths."""
    index = {c[0]: i for i, c in enumerate(code)}
    entry = {0: {}}
    work, faults = [0], set()
    starts = {0} | {index[c[3]] for c in code if c[3] is not None and c[1].startswith(("s_cbranch", "s_branch"))}
    while work:
        i = work.pop()
        state = entry[i]
        while True:
            address, mnemonic, ops, target = code[i]
            state, bad = _step(state, mnemonic, ops)
            faults.update("%x %s %s: %s" % (address, mnemonic, ", ".join(ops), b) for b in bad)
            nexts = []
            branch = mnemonic.startswith(("s_cbranch", "s_branch"))
            if branch:
                nexts.append(index[target])
            assert not mnemonic.startswith(("s_setpc", "s_swappc")), "indirect branch"
            ends = mnemonic in ("s_branch", "s_endpgm")
            if not ends:
                nexts.append(i + 1)
            through = not ends and not branch and i + 1 not in starts
            if through:
                i += 1
                continue
            for n in nexts:
                old = entry.get(n)
                new = dict(state) if old is None else {
                    k: min(a for a in (old.get(k), state.get(k)) if a is not None)
                    for k in old.keys() | state.keys()}
                if new != old:
                    entry[n] = new
                    work.append(n)
            break
    return faults


def _parse(lines):
    return [(4 * i, l.split(None, 1)[0], re.split(r",\s*(?![^\[]*\])", l.split(None, 1)[1]) if " " in l else [],
             None) for i, l in enumerate(lines)]


@pytest.mark.parametrize("lines,bad", [
    (["v_accvgpr_write_b32 a3, v1", "v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0"], True),
    (["v_accvgpr_write_b32 a3, v1", "s_nop 0", "v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0"], True),
    (["v_accvgpr_write_b32 a3, v1", "s_nop 1", "v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0"], False),
    (["v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0", "s_nop 15", "v_max_f32_e32 v20, v15, v14"], True),
    (["v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0", "s_nop 15", "s_nop 1", "v_max_f32_e32 v20, v15, v14"],
     False),
    (["v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0",
      "v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], v[0:15]"], False),
    (["v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0", "ds_write_b128 v30, v[8:11]"], True),
    (["v_mfma_f32_32x32x16_bf16 v[0:15], a[0:3], a[4:7], 0"] +
     ["v_mfma_f32_32x32x16_bf16 v[%d:%d], a[0:3], a[4:7], 0" % (16 * i, 16 * i + 15) for i in (1, 2, 3)] +
     ["v_max_f32_e32 v80, v15, v14"], False),
])
def test_the_reader_finds_planted_mistakes(lines, bad):
    code = _parse(lines + ["s_endpgm"])
    assert bool(_check(code)) == bad


def test_wait_states_of_the_built_prefill_kernels(tmp_path):
    functions = {n: c for n, c in _functions(_disassembly(tmp_path)).items() if "prefill_attn_kernel" in n}
    assert functions
    for name, code in functions.items():
        assert sum(c[1].startswith("v_mfma") for c in code) >= 32, name
        faults = _check(code)
        assert not faults, (name, len(faults), sorted(faults)[:10])


def test_wait_states_of_the_built_group_kernels(tmp_path, monkeypatch):
    """There the matrix instructions are the compiler's and only the maximum of their results is inline
    assembly, which brings its own wait.  A result of a 16x16x32 instruction (issued 4 slots after the one
    before it at the earliest) has to be 8 slots old, which is what the compiler keeps where both sides are
    its own (the kernel of 64 rows, built alike)."""
    functions = {n: c for n, c in _functions(_disassembly(tmp_path)).items() if "group_attn_kernel" in n}
    assert len(functions) == 4
    for constant, value in (("WRITE_TO_MATRIX", 0), ("MATRIX_TO_USE", 8), ("MATRIX_ISSUE", 4)):
        monkeypatch.setattr("%s.%s" % (__name__, constant), value)
    planted = _parse(["v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], 0", "s_nop 5",
                      "v_max3_f32 v20, v0, v1, v2", "s_endpgm"])
    assert _check(planted)
    for name, code in functions.items():
        assert sum(c[1].startswith("v_max3_f32") for c in code) >= 3, name
        faults = [f for f in _check(code) if "v_mfma" not in f]
        assert not faults, (name, len(faults), sorted(faults)[:10])
