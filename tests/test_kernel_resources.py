"""Registers of the kernels as built: the notes that the compiler wrote into
libgrt.so's gfx950 code objects.  The traversals run a persistent loop in which
a spilled register is stored and loaded by every step: at most four, one
16-byte access."""
import os
import re
import struct
import subprocess

import pytest

from paper_2607_22780_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{mangled kernel name: VGPRs spilled}."""
    if not os.path.exists(build.LIB):
        build.build()
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    lib = open(build.LIB, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", lib):
        at = m.start()
        (entries,) = struct.unpack_from("<Q", lib, at + 24)
        pos = at + 32
        for _ in range(entries):
            offset, size, idlen = struct.unpack_from("<QQQ", lib, pos)
            target = lib[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if not target.endswith(b"gfx950"):
                continue
            elf = tmp_path_factory.mktemp("code") / "object.elf"
            elf.write_bytes(lib[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], check=True, capture_output=True, text=True).stdout
            names = re.findall(r"^\s+\.name:\s+(_Z\S+)$", notes, re.M)
            counts = re.findall(r"^\s+\.vgpr_spill_count:\s+(\d+)$", notes, re.M)
            assert len(names) == len(counts)
            out.update(zip(names, map(int, counts)))
    return out


def test_plain_traces_do_not_spill(spills):
    trace = {n: c for n, c in spills.items() if re.match(r"_ZN3grt\d+k_traceI", n)}
    assert len(trace) == 7
    assert not {n: c for n, c in trace.items() if c > 4}


def test_backward_kernels_do_not_spill(spills):
    bwd = {n: c for n, c in spills.items() if re.match(r"_ZN3grt\d+k_(render|trace|trace_gbuffer)_bwdI", n)}
    assert len(bwd) >= 15
    assert not {n: c for n, c in bwd.items() if c > 4}
