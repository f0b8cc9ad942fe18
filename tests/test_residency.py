"""Work groups of the bf16 attention kernels that fit a compute unit at once.

The dispatch rules count on these numbers: which grids are split, and in which
order work groups are dealt, depends on how many are resident from the start.
They follow from what the compiler gave each kernel -- vector registers and
LDS, read here from the metadata of the built library's gfx950 code object --
so a change that costs a kernel its last free register shows up here."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2608_00029_amd.binding import library_path

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            p += 24
            name = blob[p:p + idlen].decode()
            p += idlen
            if "gfx950" in name:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(kernel, D, causal, parts, ragged build): (registers, LDS bytes)}; dQ's streamed form under "dq_streamed"."""
    if READELF is None:
        pytest.skip("llvm-readelf not found")
    with open(library_path(), "rb") as f:
        blob = f.read()
    out = {}
    for i, elf in enumerate(_code_objects(blob)):
        path = tmp_path_factory.mktemp("co") / f"{i}.elf"
        path.write_bytes(elf)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for k in re.split(r"\n  - \.agpr_count:", notes)[1:]:
            agpr = int(k.split()[0])
            m = re.search(r"attn_(fwd|bwd_dq|bwd_dkdv)_bf16_kernelILi(\d+)ELb([01])ELi(\d)ELi\dELb([01])E(Lb1E)?", k)
            if not m:
                continue
            name = m[1].replace("bwd_", "") + ("_streamed" if m[6] else "")
            # .vgpr_count is the total, accumulator registers included
            vgpr = int(re.search(r"\.vgpr_count:\s+(\d+)", k)[1])
            assert vgpr >= agpr
            lds = int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", k)[1])
            out[name, int(m[2]), m[3] == "1", int(m[4]), m[5] == "1"] = (vgpr, lds)
    assert out, "no bf16 attention kernels in the library's code objects"
    return out


def _per_cu(vgpr, lds):
    """A work group is four waves, one per SIMD: 512 registers a SIMD, in steps of 8; 160 KB of LDS, in steps of 1280 B."""
    return min(512 // ((vgpr + 7) // 8 * 8), 128 // ((lds + 1279) // 1280))


# work groups per CU by kernel, head dimension and parts
RESIDENT = {
    ("fwd", 64): {1: 4, 2: 3, 4: 2}, ("fwd", 128): {1: 3, 2: 2, 4: 1},
    ("dq", 64): {1: 3, 2: 2, 4: 2}, ("dq", 128): {1: 2, 2: 2, 4: 1}, ("dq_streamed", 64): {1: 4},
    ("dkdv", 64): {1: 3, 2: 2, 4: 2}, ("dkdv", 128): {1: 2, 2: 2, 4: 1},
}


@pytest.mark.parametrize("name,D", RESIDENT)
def test_resident_work_groups(kernels, name, D):
    for parts, want in RESIDENT[name, D].items():
        for causal in (True, False):
            for ragged in (True, False):
                got = kernels[name, D, causal, parts, ragged]
                assert _per_cu(*got) >= want, (name, D, "causal", causal, "parts", parts, "ragged", ragged, got)
