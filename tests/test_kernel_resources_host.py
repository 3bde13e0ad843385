"""Registers of the built round kernels, from the metadata of the device objects
that the build leaves beside the library.  A scalar that does not fit is held in
a lane of a vector register; each use then costs a vector instruction in
kernels that are bound by those, so what a round kernel specialized for a
quantizer with codes of its own spills is bounded.  (With the row descriptors'
masks and the server's arguments held through the workers' side these kernels
spilled 20 to 629 scalars, and Example 1 in wide buckets took a sixth longer.)"""
import glob
import os
import re
import struct
import subprocess

import pytest

BUILD = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2205_14473_amd", "_build")
READELF = "/opt/rocm/lib/llvm/bin/llvm-readelf"
OBJECTS = sorted(glob.glob(os.path.join(BUILD, "ea_*.hip.hipfb")))

pytestmark = pytest.mark.skipif(not OBJECTS or not os.path.exists(READELF), reason="no device objects or no readelf here")

Q_TOPK = 5
MOST_SPILLED = 48       # the worst of these kernels spills 35, the BERT-sized round's 6


def _device_code(path):
    """The gfx950 entry of a clang offload bundle."""
    with open(path, "rb") as f:
        b = f.read()
    assert b[:24] == b"__CLANG_OFFLOAD_BUNDLE__", path
    at = 32
    for _ in range(struct.unpack_from("<Q", b, 24)[0]):
        off, size, n = struct.unpack_from("<QQQ", b, at)
        if b"gfx950" in b[at + 24:at + 24 + n]:
            return b[off:off + size]
        at += 24 + n
    raise AssertionError(f"{path}: no gfx950 code")


def _round_kernels(path, tmp_path):
    """(worker quantizer's kind, scalars spilled, name) of each step_kernel with a fixed worker quantizer."""
    elf = tmp_path / "code"
    elf.write_bytes(_device_code(path))
    notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
    for entry in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
        name = re.search(r"\.symbol:\s+'?(\S+?)'?\s", entry).group(1)
        m = re.search(r"step_kernelILi\dENS_3QCtILi(\d+)E", name)
        if m:
            yield int(m.group(1)), int(re.search(r"\.sgpr_spill_count:\s+(\d+)", entry).group(1)), name


def test_round_kernels_hold_their_scalars(tmp_path):
    seen, bad = 0, []
    for path in OBJECTS:
        for kind, spilled, name in _round_kernels(path, tmp_path):
            if kind < Q_TOPK:
                seen += 1
                if spilled > MOST_SPILLED:
                    bad.append((spilled, name))
    assert seen > 50, "round kernels not found"
    assert not bad, bad
