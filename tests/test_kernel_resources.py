"""What the compiler gave the kernels of the built library, from the metadata of its code objects
(no GPU needed): no kernel spills vector registers or uses scratch memory, and the decoder's variants leave
room for as many workgroups a compute unit as their launch bounds name."""
import os
import re
import struct
import subprocess

import pytest

import paper_2411_19114_amd as prep

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
LDS, LDS_UNIT, VGPRS = 160 << 10, 1280, 512   # of a compute unit; what LDS is given out in; of a SIMD's lane


def _code_objects(path):
    """The gfx950 ELF images in the library's offload bundles."""
    data = open(path, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.end()
        n, = struct.unpack_from("<Q", data, at)
        at += 8
        if n > 16:
            continue   # (the text itself, not a bundle)
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in name and size:
                yield data[m.start() + off:m.start() + off + size]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(prep.lib_path()):
        prep.build()
    found = {}
    for i, elf in enumerate(_code_objects(prep.lib_path())):
        p = tmp_path_factory.mktemp("co") / f"{i}.elf"
        p.write_bytes(elf)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True, check=True).stdout
        for k in re.split(r"^  - ", notes, flags=re.M)[1:]:
            fields = dict(re.findall(r"^ {4}\.(\w+): +(\S+)$", k, flags=re.M))
            if "name" in fields:
                found[fields["name"]] = fields
    return found


def test_no_kernel_spills(kernels):
    assert len(kernels) >= 10
    for name, k in kernels.items():
        assert int(k["vgpr_spill_count"]) == 0 and int(k["private_segment_fixed_size"]) == 0, name


# decode_entropy<hypotheses, run entries>
@pytest.mark.parametrize("variant,want", [("ILb1ELb1E", 3), ("ILb0ELb1E", 3), ("ILb0ELb0E", 4)])
def test_workgroups_of_the_decoder_a_compute_unit(kernels, variant, want):
    (k,) = [v for n, v in kernels.items() if "decode_entropy" + variant in n]
    assert LDS // (-(-int(k["group_segment_fixed_size"]) // LDS_UNIT) * LDS_UNIT) >= want
    assert VGPRS // (-(-int(k["vgpr_count"]) // 8) * 8) >= want   # a workgroup has a wave on every SIMD
