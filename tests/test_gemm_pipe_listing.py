"""The large GEMM writes its accumulators from inline assembly, whose latency the compiler does not know.  This test compiles
the kernel and checks, instruction by instruction, that the compiled code keeps the wait states the hardware asks for: no
accumulator is touched by anything but an MFMA before the MFMA that wrote it is done, no MFMA reads a register right behind
the vector instruction that wrote it, and no fetch reads a scalar register right behind a vector write of it.  The last holds for every kernel
that fetches straight into LDS from inline assembly."""
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from listing import listing

FETCHING = ("attention_mfma", "gemm_codes", "gemm_fit", "gemm_fit_int8", "gemm_ring", "gemm_stream", "ordered_kernels")

MFMA = "v_mfma_f32_16x16x32_bf16"
RESULT_STATES = 12          # 8-pass MFMA result -> vector ALU or LDS read: 11 wait states
SOURCE_STATES = 2           # vector ALU result -> MFMA source
SCALAR_STATES = 5           # vector ALU result in an SGPR -> memory instruction


def _regs(text, kind):
    out = set()
    for lo, hi, one in re.findall(rf"\b{kind}\[(\d+):(\d+)\]|\b{kind}(\d+)\b", text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def _kernels(text):
    for m in re.finditer(r"^(_Z\S*kernel\S*):", text, re.M):
        body = text[m.end():]
        lines, inline = [], False
        for raw in body[:body.index(".Lfunc_end")].splitlines():
            inline = (inline or "#ASMSTART" in raw) and "#ASMEND" not in raw
            line = raw.split(";")[0].strip()
            if line and not line.endswith(":") and not line.startswith("."):
                lines.append(("asm " if inline and line.startswith("v_mfma") else "") + line)
        yield m.group(1), lines


def _violations(lines):
    """Straight-line scan; "asm " marks the MFMAs whose results the compiler knows nothing about (it takes care of its own)."""
    written, vector, scalar, found = [], [], [], []
    for line in lines:
        opaque = line.startswith("asm ")
        op, _, args = (line[4:] if opaque else line).partition(" ")
        dst = args.split(",")[0]
        states = int(args) + 1 if op == "s_nop" else 4 if op.startswith("v_mfma") else 1
        if op.startswith("v_mfma"):
            src = _regs(args, "v"), _regs(args, "a")
            found += [line for v, a, age in vector if age < SOURCE_STATES and (v & src[0] or a & src[1])]
        elif _regs(args, "a"):
            found += [line for a, age in written if age < RESULT_STATES and a & _regs(args, "a")]
        if "offen lds" in line:
            found += [line for s, age in scalar if age < SCALAR_STATES and s & _regs(args, "s")]
        written = [(a, n + states) for a, n in written if n < 40]
        vector = [(v, a, n + states) for v, a, n in vector if n < 8]
        scalar = [(s, n + states) for s, n in scalar if n < 8]
        if opaque:
            written.append((_regs(dst, "a"), 0))
        elif op in ("v_readlane_b32", "v_readfirstlane_b32") or op.startswith("v_cmp"):
            scalar.append((_regs(dst, "s"), 0))
        elif op.startswith("v_") and not op.startswith("v_mfma"):
            vector.append((_regs(dst, "v"), _regs(dst, "a"), 0))
    return found


@pytest.fixture(scope="module", autouse=True)
def _compiled():
    with ThreadPoolExecutor(4) as ex:
        list(ex.map(listing, ("gemm_pipe",) + FETCHING))


def test_compiled_gemm_keeps_its_wait_states():
    kernels = [k for k in _kernels(listing("gemm_pipe")) if "gemm_pipe_kernel" in k[0]]
    assert len(kernels) >= 20
    for name, lines in kernels:
        assert sum(l.startswith("asm " + MFMA) for l in lines) >= 256, name
        assert not _violations(lines), (name, _violations(lines)[:3])


@pytest.mark.parametrize("source", FETCHING)
def test_fetches_wait_for_their_scalars(source):
    fetching = [(n, lines) for n, lines in _kernels(listing(source)) if any("offen lds" in l for l in lines)]
    assert fetching
    for name, lines in fetching:
        for i, line in enumerate(lines):
            if "offen lds" in line:                        # the LDS address, one wait state or more, the fetch
                assert lines[i - 1].startswith("s_nop") and lines[i - 2].startswith("s_mov_b32 m0,"), (name, lines[i - 2:i + 1])
        assert not _violations(lines), (name, _violations(lines)[:3])


def test_scan_sees_a_hazard():
    bad = [f"asm {MFMA} a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 3", "v_accvgpr_read_b32 v9, a2"]
    assert _violations(bad) and not _violations([bad[0], "s_nop 15", bad[2]])
    assert _violations(["v_accvgpr_write_b32 a1, v2", bad[0]]) and not _violations(["v_accvgpr_write_b32 a1, v2", "s_nop 1", bad[0]])
    fetch = "buffer_load_dwordx4 v1, s[0:3], s9 offen lds"
    assert _violations(["v_readlane_b32 s9, v1, 0", fetch]) and not _violations(["v_readlane_b32 s9, v1, 0", "s_nop 4", fetch])
