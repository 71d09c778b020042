"""Registers of the built kernels, from the code objects inside libmira.so: the
occupancies that the tile shapes and dispatch rules count on, and no vector
registers spilled."""
import os
import re
import struct
import subprocess

import pytest

import paper_2609_38090_amd as mira

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: {field: value}} of every gfx950 code object in the library."""
    lib = os.path.join(os.path.dirname(mira.__file__), "libmira.so")
    if not os.path.exists(lib) or not os.path.exists(READELF):
        pytest.skip("no built library or no llvm-readelf")
    with open(lib, "rb") as f:
        data = f.read()
    tmp, found = tmp_path_factory.mktemp("code"), {}
    # offload bundles: magic, entry count, then (offset, size, id length, id) each
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.end()
        n, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" not in name or not size:
                continue
            path = tmp / f"{m.start()}.co"
            path.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - (?=\.)", notes)[1:]:
                fields = dict(re.findall(r"^ *(\.\w+): +(\S+)$", k, re.M))
                if ".vgpr_count" in fields and ".symbol" in fields:
                    found[fields[".symbol"]] = fields
    assert found
    return found


def _vgprs(kernels, part):
    hit = [int(v[".vgpr_count"]) for k, v in kernels.items() if part in k]
    assert hit, part
    return max(hit)


def test_no_vector_spills(kernels):
    assert not [k for k, v in kernels.items() if int(v[".vgpr_spill_count"])]


# 512 registers per SIMD lane, in blocks of 8: 256 for two waves, 168 for three
@pytest.mark.parametrize("part,most", [
    # narrow prefill down tiles: two workgroups of four waves per CU
    ("prefill_gemm_kernelILb0ELi2E", 256),
    # INT8 gate/up of two and three token groups at small hidden sizes: three
    # workgroups of four waves per CU
    ("decode_gateup_kernelILi2ELb0ELi3E", 168),
    ("decode_gateup_kernelILi3ELb0ELi3E", 168),
])
def test_occupancy(kernels, part, most):
    assert _vgprs(kernels, part) <= most
