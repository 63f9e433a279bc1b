"""Registers and LDS of the built kernels, where the launch rules count on an
occupancy.  Read from the metadata of the code objects in libmppi.so."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

from paper_2509_14726_amd import build as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LDS_PER_CU, VGPRS_PER_SIMD = 160 * 1024, 512


def _code_objects(data):
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        o = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, o)
            if size and b"gfx" in data[o + 24:o + 24 + n]:
                yield data[at + off:at + off + size]
            o += 24 + n
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels():
    """Name (template arguments as mangled) -> integer fields of its metadata."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    out = {}
    for obj in _code_objects(open(B.LIB, "rb").read()):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            fields = {k: int(v) for k, v in re.findall(r"\.([a-z_]+):\s+(\d+)\s*$", block, flags=re.M)}
            out[re.search(r"\.name:\s+(\S+)", block)[1]] = fields
    assert out
    return out


def matching(kernels, pattern):
    found = {k: v for k, v in kernels.items() if re.search(pattern, k)}
    assert found, pattern
    return found


def waves_per_simd(k):
    return min(8, VGPRS_PER_SIMD // ((k["vgpr_count"] + 7) // 8 * 8))


@pytest.mark.parametrize("objective", [0, 1, 2])
def test_two_pipelines_with_short_rings_share_a_cu(kernels, objective):
    """Binary32 pipelines with rings of 4 steps, alone and batched: the launch
    rules count two workgroups per CU."""
    for k in matching(kernels, r"kb?_rollout4ILi%dEfLi4E" % objective).values():
        waves = k["max_flat_workgroup_size"] // 64
        assert 4 * waves_per_simd(k) >= 2 * waves
        assert 2 * k["group_segment_fixed_size"] <= LDS_PER_CU


@pytest.mark.parametrize("pipe,rate", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("objective", [0, 1, 2])
def test_batched_drawing_rollouts_spill_nothing(kernels, objective, pipe, rate):
    """A spilled value would be read behind the sample's store in every step.
    The grid counts three (two with PIPE or the rate input) waves per SIMD."""
    for k in matching(kernels, r"kb_rollout_drawILi%dEfLb%dELb%dELb[01]E" % (objective, pipe, rate)).values():
        assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0
        assert waves_per_simd(k) >= (2 if pipe or rate else 3)


def test_no_kernels_that_nothing_launches(kernels):
    """Binary64 samples always take binary64 sums, and rounds of loads; all of a
    thread's samples at once are loaded up to 8192 binary32 samples, below the
    65536 from which sums are binary64."""
    assert not [k for k in kernels if re.search(r"k_finalId[^d]|kb_finalId[^d]", k)]
    assert not [k for k in kernels if re.search(r"k_finalI(d|fd).*Li8E", k)]
