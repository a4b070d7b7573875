"""The LDS swizzles of the kernels on the CPU, from the expressions of the
source file: bank conflicts of the fragment reads and the copies that fill
the rows."""
import os
import re

import pytest

from paper_2605_01060_amd import build as B

with open(os.path.join(B.CSRC, "device_common.h")) as _f:
    SRC = _f.read()

# Lanes of a half wave that a 16-byte read is served for at once.
FIRST = [*range(0, 4), *range(12, 16), *range(20, 28)]
GROUPS = [FIRST, [lane for lane in range(32) if lane not in FIRST]]


def _expression(pattern):
    return re.search(pattern, SRC).group(1).replace("/", "//")


ROWS32 = _expression(r"if \(CPR == 8\) return (row \* 8 \+ .*?);")
ROWS16 = _expression(r"int swz16\(int row, int chunk\) \{\s*return (.*?);")
COPY32 = _expression(r"if \(CPR == 8\) return (\(lane & 7\) .*?);")
COPY16 = _expression(r"int copy_chunk16\(int lane\) \{ return (.*?); \}")


def _slot(expr, row, chunk):
    return eval(expr, {"row": row, "chunk": chunk})


@pytest.mark.parametrize("ks", range(4))
def test_reads_of_32_rows_have_no_bank_conflicts(ks):
    for half in range(2):
        for lanes in GROUPS:
            slots = {_slot(ROWS32, lane, 2 * ks + half) % 16 for lane in lanes}
            assert len(slots) == 16


@pytest.mark.parametrize("ks", range(2))
def test_reads_of_16_rows_and_4_chunks_have_no_bank_conflicts(ks):
    for half in range(2):
        for lanes in GROUPS:
            slots = {_slot(ROWS16, lane % 16, 4 * ks + 2 * half + lane // 16) % 16
                     for lane in lanes}
            assert len(slots) == 16


@pytest.mark.parametrize("swizzle,copy_chunk", [(ROWS32, COPY32), (ROWS16, COPY16)])
def test_a_copy_puts_each_chunk_where_it_is_read(swizzle, copy_chunk):
    """Copy j fills rows 8 j .. 8 j + 7 with 64 consecutive slots."""
    for copy in range(4):
        for lane in range(64):
            chunk = eval(copy_chunk, {"lane": lane, "copy": copy})
            assert _slot(swizzle, 8 * copy + lane // 8, chunk) == 64 * copy + lane


def test_the_second_k_steps_chunks_differ_in_one_bit():
    """linear_wide.hip reads K step 1 at the address of K step 0 ^ 64."""
    for row in range(16):
        for chunk in range(4):
            assert _slot(ROWS16, row, chunk + 4) * 16 == (_slot(ROWS16, row, chunk) * 16) ^ 64
