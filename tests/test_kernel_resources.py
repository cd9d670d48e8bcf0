"""Registers of the encoder kernels, from the metadata of the built library's own code objects (no GPU): a kernel that is
launched for two workgroups per CU, two wavefronts per SIMD, must fit twice into a SIMD's 512 registers a lane, or its
second workgroup never becomes resident."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

from paper_1803_09877_amd import binding as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 code objects of a host library: each offload bundle lists (offset, size, target) entries."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(min(count, 16)):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len]
            entry += 24 + name_len
            if b"gfx950" in name and size > 0:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels():
    """{mangled kernel name: (registers incl. accumulation registers, scratch bytes)}"""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    B.lib()
    out = {}
    with open(B.LIB_PATH, "rb") as f:
        blob = f.read()
    for obj in code_objects(blob):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for part in notes.split("- .agpr_count:")[1:]:
            field = {k: v for k, v in re.findall(r"^\s+(\.\w+):\s+(\S+)$", "    .agpr_count: " + part.lstrip(), re.M)}
            out[field[".name"]] = (int(field[".vgpr_count"]), int(field[".private_segment_fixed_size"]))
    return out


def arguments(kernels, name):
    """{template arguments, as numbers: what `kernels` holds} of the kernel templates of this name."""
    found = {}
    for k, v in kernels.items():
        m = re.search(rf"{len(name)}{name}I((?:L[ib]\d+E)+)E", k)
        if m:
            found[tuple(int(n) for n in re.findall(r"L[ib](\d+)E", m.group(1)))] = v
    return found


def test_unpacked_encoders_fit_as_often_as_they_are_launched(kernels):
    found = arguments(kernels, "encode_cyc_real_kernel")
    for (s, _, _, per_cu), (registers, scratch) in found.items():
        assert registers <= 512 // per_cu, (s, per_cu, registers)
        assert scratch == 0 or (s, per_cu) == (8, 2), (s, per_cu, scratch)
    assert {s for s, _, _, per_cu in found if per_cu == 2} == set(range(9))


def test_packed_encoders_fit_as_often_as_they_are_launched(kernels):
    ring, rounds = (arguments(kernels, "encode_cyc" + n + "_kernel") for n in ("", "_rounds"))
    for (s, *_, per_cu), (registers, scratch) in list(ring.items()) + list(rounds.items()):
        assert registers <= 512 // per_cu, (s, per_cu, registers)
        assert scratch <= (64 if (s, per_cu) == (7, 2) else 0), (s, per_cu, scratch)
    for found, widest in ((ring, 7), (rounds, 7)):
        assert {s for s, *_, per_cu in found if per_cu == 2} == set(range(widest + 1))


def test_locators_that_recombine_keep_their_rows_in_registers(kernels):
    """Two wavefronts per SIMD: a workgroup of eight (short rows), two workgroups of four (longer ones).  Rows in flight that
    spill go through memory and back while the locator runs."""
    short, walk = (arguments(kernels, "cyc_locate_" + n + "_kernel") for n in ("recombine", "walk"))
    assert {lo for lo, _ in short} == {lo for lo, _ in walk} and {chunks for _, chunks in short} == {1, 2, 4}
    for form, (registers, scratch) in list(short.items()) + list(walk.items()):
        assert registers <= 256 and scratch == 0, (form, registers, scratch)
