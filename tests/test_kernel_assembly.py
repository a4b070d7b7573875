"""What the compiler made of the kernels, from its assembly.

The linear kernels wait for their inline-assembly copies themselves; the
compiler does not know of those copies.  A register that it spills inside
them comes back with a wait of the compiler's own, which drains every copy in
flight.
"""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2605_01060_amd import build as B


def _assembly(src):
    cmd = [B.hipcc(), "-x", "hip", "-S", "--offload-device-only", src, "-o", "-"] \
        + B.COMMON + B.HIP_FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


@pytest.fixture(scope="module")
def assembly():
    try:
        B.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    srcs = [s for s in B.sources() if s.endswith(".hip")]
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        return dict(zip(map(os.path.basename, srcs), ex.map(_assembly, srcs)))


def _kernels(text):
    """(name, resources, body) of every kernel of a source's assembly."""
    for block in re.split(r"\n  - \.agpr_count", text)[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        res = {k: int(re.search(rf"\.{k}:\s+(\d+)", block).group(1))
               for k in ("vgpr_spill_count", "private_segment_fixed_size")}
        start = text.index(f"\n{name}:")
        yield name, res, text[start:text.index(".Lfunc_end", start)]


def test_no_kernel_spills(assembly):
    found = 0
    for src, text in assembly.items():
        for name, res, _ in _kernels(text):
            found += 1
            assert not any(res.values()), (src, name, res)
    assert found >= 60


def test_no_wait_of_the_compilers_between_the_wide_tiles_mfmas(assembly):
    """Every basic block with MFMAs waits for vector memory only where the
    kernel says so, in inline assembly."""
    checked = 0
    for name, _, body in _kernels(assembly["linear_wide.hip"]):
        mfmas, waits, inline = 0, 0, False
        for line in body.split("\n") + [".LBB_end:"]:
            op = line.strip()
            if op.startswith(".LBB"):
                assert not (mfmas and waits), (name, mfmas, waits)
                checked += mfmas
                mfmas = waits = 0
            inline = op == ";;#ASMSTART" or (inline and op != ";;#ASMEND")
            mfmas += op.startswith("v_mfma")
            waits += not inline and op.startswith("s_waitcnt") and "vmcnt" in op
    assert checked >= 14 * 48


def test_nothing_before_the_128_wide_tiles_copies(assembly):
    """In the K loop the barrier that frees a stage's buffer is followed by
    the copies into it, with no MFMAs to issue first."""
    loops = 0
    for name, _, body in _kernels(assembly["linear.hip"]):
        for block in body.split("\n.LBB"):
            lines = [line.strip() for line in block.split("\n")]
            if not any(op.startswith("v_mfma") for op in lines) or "s_barrier" not in lines:
                continue
            after = lines[lines.index("s_barrier"):]
            copy = next(i for i, op in enumerate(after) if op.startswith("global_load_lds"))
            assert not any(op.startswith("v_mfma") for op in after[:copy]), name
            loops += 1
    assert loops >= 10
