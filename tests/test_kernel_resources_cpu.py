"""Register and LDS use of the kernels that are sized to fit a fixed number of
work-groups on a CU, read from the code-object metadata of the built library
(no GPU needed).  CPU only."""
from __future__ import annotations

import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1102_1343_amd", "libfire_gfx950.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of the offload bundles in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        o = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", blob, o)
        o += 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, o)
            if b"gfx950" in blob[o + 24:o + 24 + ln] and size:
                yield blob[at + off:at + off + size]
            o += 24 + ln
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Metadata of every kernel, keyed by mangled name."""
    if not os.path.exists(LIB):
        pytest.skip("library not built (run __graft_entry__.build())")
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    out = {}
    for co in _code_objects(open(LIB, "rb").read()):
        p = tmp_path_factory.mktemp("co") / "co.elf"
        p.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True,
                               check=True).stdout
        for part in notes.split("\n  - .agpr_count:")[1:]:
            d = dict(re.findall(r"^    \.(\w+): +(\S+)$", part, re.M))
            out[d["name"]] = {k: int(v) for k, v in d.items() if v.isdigit()}
    assert len(out) > 50
    return out


def _one(kernels, name):
    hit = [v for k, v in kernels.items() if name in k]
    assert len(hit) == 1, (name, len(hit))
    return hit[0]


def test_default_step_has_registers_for_four_work_groups(kernels):
    """The FP32 120 x 20 step: 8 waves per SIMD take at most 64 vector
    registers; nothing in scratch, and few scalar spills (values used once, in
    the ignition set-up and at the domain's edge: row numbers and masks that
    live across the kernel's phases give 28 and more)."""
    k = _one(kernels, "k_stepIfLi7ELb1ELb0ELb0EE")
    assert k["vgpr_count"] <= 64
    assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0
    assert k["sgpr_spill_count"] <= 12


@pytest.mark.parametrize("name,groups,row", [("k_stepIfLi7ELb1ELb0ELb0EE", 4, 48),
                                             ("k_stepIdLi7ELb1ELb0ELb0EE", 2, 96)])
def test_step_lds_with_21_fuels(kernels, name, groups, row):
    """A CU's 160 KiB hold four FP32 (two FP64) 120 x 20 work-groups with the
    rows of 21 fuels and the activity word behind the frames."""
    k = _one(kernels, name)
    assert groups * (k["group_segment_fixed_size"] + 21 * row + 4) <= 160 * 1024


@pytest.mark.parametrize("name", ["k_stepIfLi7ELb1ELb0ELb1EE", "k_ens_stepIfLi7ELb1EE"])
def test_few_tiles_and_ensembles_have_registers_for_three_work_groups(kernels, name):
    """FP32 120 x 20 tiles, three work-groups (24 waves) on a CU: at most 80
    vector registers, no scratch, and the wave's row in a vector register, so
    no scalar spills."""
    k = _one(kernels, name)
    assert k["vgpr_count"] <= 80
    assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0
    assert k["sgpr_spill_count"] == 0


def test_small_tile_kernels_that_no_rule_launches_are_not_built(kernels):
    """FP64 small tiles have at most 1024 nodes, one per thread."""
    small = [k for k in kernels if "k_step_small" in k or "k_ens_small" in k]
    assert len(small) == 9
    assert not [k for k in small if "smallIdLi2E" in k or "smallIdLb0ELi2E" in k
                or "smallIdLb1ELi2E" in k]
