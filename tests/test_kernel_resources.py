"""Registers of the built kernels where a rule or a launch shape counts on how
many waves a SIMD (512 registers) holds, from the metadata of this build's own
library (no GPU needed)."""
import re
import struct
import subprocess
from pathlib import Path

import pytest

from paper_1004_1932_amd import build

READELF = Path("/opt/rocm/llvm/bin/llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled-enough name: metadata} of every kernel in libad.so."""
    if not READELF.exists():
        pytest.skip("needs ROCm's llvm-readelf")
    if not build.LIB.exists():
        build.build()
    blob, out, at = build.LIB.read_bytes(), {}, 0
    while (at := blob.find(MAGIC, at)) >= 0:
        count, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"amdgcn" in name and size:
                f = tmp_path_factory.mktemp("code") / "code.o"
                f.write_bytes(blob[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", f], capture_output=True, text=True, check=True).stdout
                for block in notes.split("- .agpr_count")[1:]:
                    sym = re.search(r"\.symbol:\s+'?(\S+?)\.kd", block)
                    out[sym.group(1)] = {k: int(v) for k, v in re.findall(
                        r"\.(vgpr_count|vgpr_spill_count|private_segment_fixed_size):\s+(\d+)", block)}
        at += len(MAGIC)
    assert out
    return out


def _of(kernels, name, *args):
    """Metadata of the instances whose first template arguments are args (None: any)."""
    pat = re.compile(rf"^_ZN2ad\d+{name}I" + "".join(r"Li\d+E" if a is None else rf"Li{a}E" for a in args))
    found = {k: v for k, v in kernels.items() if pat.match(k)}
    assert found, (name, args)
    return found


def _waves(v):
    """Waves per SIMD that the registers (allocated by eights) allow."""
    return min(8, 512 // ((v["vgpr_count"] + 7) // 8 * 8))


def test_fused_stage_of_ensembles_holds_six_waves(kernels):
    """Its many work-groups of four waves hide each other's latencies."""
    for k, v in _of(kernels, "k_stage_fused", None, None, 4).items():
        assert _waves(v) >= 6 and v["vgpr_spill_count"] == 0, (k, v)


@pytest.mark.parametrize("targets", [4, 8])
def test_streamed_stage_of_eight_waves_shares_a_compute_unit(kernels, targets):
    """Two work-groups of eight waves on a compute unit's four SIMDs, which from
    2048 to 4095 spheres it is chosen for."""
    for k, v in _of(kernels, "k_stage_stream", None, None, targets, 8, None).items():
        assert _waves(v) >= 4 and v["vgpr_spill_count"] == 0, (k, v)


def test_pair_kernel_of_four_targets_per_lane_holds_four_waves(kernels):
    for k, v in _of(kernels, "k_pairs_f32c", None, 4, None, None, 0, None).items():
        assert _waves(v) >= 4 and v["vgpr_spill_count"] == 0, (k, v)


def test_resident_kernels_hold_the_work_groups_their_rule_counts_on(kernels):
    """The table in resident_one: work-groups per compute unit (one wave per
    SIMD each) with and without the form of up to 16 spheres."""
    src = (build.CSRC / "ad_kernels.hip").read_text()
    rows = re.search(r"with\[2\]\[3\] = \{\{(.*?)\}, \{(.*?)\}\}, without\[2\]\[3\] = \{\{(.*?)\}, \{(.*?)\}\};", src)
    table = [[int(x) for x in r.split(",")] for r in rows.groups()]
    for one in (1, 0):
        for rpy in (0, 1):
            for integ in range(3):
                (v,) = _of(kernels, "k_resident", rpy, integ, one).values()
                assert _waves(v) == table[2 * (1 - one) + rpy][integ], (rpy, integ, one, v)
