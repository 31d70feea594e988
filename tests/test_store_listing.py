"""Stores of 16 bytes read their last registers some cycles after they were issued, and the compiler waits for that only where the scalar
offset of the store is no register.  This test compiles the kernels that store accumulators through buffers and checks that form and
the wait."""
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from listing import listing

SOURCES = ("gemm_codes", "gemm_pipe", "gemm_fit", "gemm_fit_int8")
WAIT_STATES = 2
STORE = re.compile(r"buffer_store_dwordx([34]) v\[(\d+):(\d+)\], (?:v\d+|off), s\[\d+:\d+\], (\S+)")


def _violations(lines):
    data, found = [], []                                  # (registers of a store, wait states since)
    for line in lines:
        op, _, args = line.partition(" ")
        if op.startswith("v_"):                            # (loads return long after)
            dst = args.split(",")[0]
            m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)$", dst)
            if m:
                regs = {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))
                found += [line for r, age in data if age < WAIT_STATES and r & regs]
        data = [(r, age + (int(args) + 1 if op == "s_nop" else 1)) for r, age in data if age < 8]
        m = STORE.match(line)
        if m:
            if m[4] != "0":
                found.append(line)
            data.append((set(range(int(m[2]), int(m[3]) + 1)), 0))
    return found


@pytest.fixture(scope="module", autouse=True)
def _compiled():
    with ThreadPoolExecutor(4) as ex:
        list(ex.map(listing, SOURCES))


@pytest.mark.parametrize("name", SOURCES)
def test_stores_wait_for_their_data(name):
    lines = [l.split(";")[0].strip() for l in listing(name).splitlines()]
    lines = [l for l in lines if l and not l.startswith(".") and not l.endswith(":")]
    assert sum(bool(STORE.match(l)) for l in lines) >= 64
    assert not _violations(lines), _violations(lines)[:3]


def test_scan_sees_both_faults():
    store = "buffer_store_dwordx4 v[4:7], v0, s[16:19], 0 offen"
    assert not _violations([store, "s_nop 1", "v_mov_b32_e32 v7, 0"]) and not _violations([store, "v_mov_b32_e32 v8, 0"])
    assert _violations([store, "v_mov_b32_e32 v7, 0"]) and _violations([store, "s_nop 0", "v_mov_b32_e32 v4, 0"])
    assert _violations([store.replace(", 0 offen", ", s20 offen")])
