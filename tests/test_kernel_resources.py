"""Registers and scratch of the built kernels, from the metadata of the
library's own code objects: a change that costs a kernel its workgroups per
compute unit, or makes it spill, shows here without a GPU.

A gfx950 SIMD has 512 vector registers per lane, given out in eights; a
compute unit has four SIMDs.
"""
import re
import struct
import subprocess
import tempfile

import pytest

from paper_2110_07670_amd import _lib, build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(data):
    """The gfx950 code objects of a shared library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", data, at + len(magic))
        q = at + len(magic) + 8
        for _ in range(count):
            off, size, tl = struct.unpack_from("<QQQ", data, q)
            if b"gfx950" in data[q + 24:q + 24 + tl]:
                yield data[at + off:at + off + size]
            q += 24 + tl
        at += len(magic)


@pytest.fixture(scope="module")
def kernels():
    """(name, type, template numbers) -> (registers, scratch bytes, threads)."""
    _lib.load()
    found = {}
    with open(build.LIB, "rb") as f:
        data = f.read()
    for obj in _code_objects(data):
        with tempfile.NamedTemporaryFile(suffix=".co") as t:
            t.write(obj)
            t.flush()
            text = subprocess.run([READELF, "--notes", t.name], capture_output=True, text=True,
                                  check=True).stdout
        for part in re.split(r"\n  - \.agpr_count", text)[1:]:
            get = lambda key: re.search(r"\.%s:\s+(\S+)" % key, part).group(1)  # noqa: E731
            m = re.match(r"_ZN4acex\d+(k_\w+?)I([df])((?:L[ib]\d+E)+)E", get("symbol"))
            if m:
                args = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(3)))
                found[m.group(1), m.group(2), args] = (
                    int(get("vgpr_count")), int(get("private_segment_fixed_size")),
                    int(get("max_flat_workgroup_size")))
    return found


def _waves(regs):
    """Waves per SIMD that the registers leave."""
    return min(8, 512 // (-(-regs // 8) * 8))


def test_four_pass_update_keeps_its_waves(kernels):
    """The W update of full tiles in the four-pass schedule: three waves per
    SIMD, two in the FP32 form of 16 orbitals off the diagonal."""
    got = {k: v for k, v in kernels.items() if k[0] == "k_accumulate_full"}
    assert got
    for name, (regs, scratch, _) in got.items():
        assert scratch == 0, (name, scratch)
        assert _waves(regs) >= (2 if name[1:] in {("f", (16, 0, 0)), ("f", (16, 0, 1))} else 3), \
            (name, regs)


def _groups(regs, threads):
    """Workgroups per compute unit that the registers leave."""
    return 4 * _waves(regs) // (threads // 64)


def test_batch_pass_keeps_its_workgroups(kernels):
    """The persistent inverse-z/W pass fits as many workgroups as the
    single-system kernels whose work it does (but for 48^3 FP64 in blocks of 8,
    98 registers against 92: two for three)."""
    got = [k for k in kernels if k[0] == "k_batch_pass" and k[2][0] == 2]
    assert got
    for name in got:
        _, n, block = name[2]
        if name[1:] == ("d", (2, 48, 8)):
            continue
        own = [kernels["k_zinv_acc", name[1], (n, block, diag, 0)] for diag in (0, 1)]
        want = min(_groups(regs, threads) for regs, _, threads in own)
        regs, _, threads = kernels[name]
        assert _groups(regs, threads) >= want, (name, regs, own)


def test_slab_forward_has_no_scratch(kernels):
    got = {k: v for k, v in kernels.items() if k[0] == "k_slab_fwd"}
    assert got
    for name, (_, scratch, _) in got.items():
        assert scratch == 0, (name, scratch)


def test_incomplete_tile_kernels_are_reached(kernels):
    """The fused pass of incomplete tiles is compiled for the grids that take it."""
    grids = {t: {k[2][0] for k in kernels if k[0] == "k_zinv_list" and k[1] == t} for t in "df"}
    assert grids["d"] == {16, 24, 32, 40, 48, 64, 80, 96, 120}
    assert grids["f"] == {40, 48, 64, 80, 96, 128}
