"""Scratch (spilled registers) of the built kernels, from the code object's own
metadata: what the large calls run keeps to the figures it was measured with."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
BF16, TENSOR, ROW, MX = 0, 1, 2, 3
SCORE, DRAW, DZ, PRODUCT, LOGITS, MEASURES = range(6)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{(mode, epilogue, waves, token blocks, persistent, row-major W): bytes of scratch per lane} of score_kernel."""
    from paper_2607_24062_amd import acrl
    if not os.path.exists(acrl.LIB_PATH) or not os.path.exists(READELF):
        pytest.skip("no built library or no llvm-readelf")
    with open(acrl.LIB_PATH, "rb") as f:
        lib = f.read()
    got = {}
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", lib):  # magic, count, then (offset, size, triple length, triple)
        at = m.end()
        (n,) = struct.unpack_from("<Q", lib, at)
        at += 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", lib, at)
            triple = lib[at + 24:at + 24 + tl]
            at += 24 + tl
            if b"gfx950" not in triple or not size:
                continue
            path = tmp_path_factory.mktemp("co") / "k.co"
            path.write_bytes(lib[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - ", notes):
                name = re.search(r"\.name:\s+\S*score_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)E", k)
                size_of = re.search(r"\.private_segment_fixed_size:\s+(\d+)", k)
                if name and size_of:
                    got[tuple(int(x) for x in name.groups())] = int(size_of.group(1))
    assert got, "no score kernel found in the library"
    return got


@pytest.mark.parametrize("mode,most", [(BF16, 0), (TENSOR, 28), (ROW, 12)])
def test_packed_scorers(scratch, mode, most):
    assert scratch[mode, SCORE, 8, 2, 1, 0] <= most


@pytest.mark.parametrize("key,most", [((TENSOR, LOGITS, 8, 2, 1, 0), 40), ((ROW, LOGITS, 8, 2, 0, 0), 40),
                                      ((MX, LOGITS, 4, 4, 1, 0), 0), ((BF16, MEASURES, 8, 2, 1, 0), 12)])
def test_packed_measures(scratch, key, most):
    assert scratch[key] <= most


def test_no_scratch_elsewhere(scratch):
    narrow = [k for k in scratch if 16 * k[2] * k[3] < 256]
    others = [k for k in scratch if k[1] in (DRAW, DZ, PRODUCT) or (k[1] == SCORE and k[0] == MX)]
    assert narrow and others
    assert {k: scratch[k] for k in narrow + others if scratch[k]} == {}
