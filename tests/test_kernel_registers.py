"""Registers of the stencil kernels in the built library, from the metadata that the
compiler leaves beside each kernel: a wavefront's 512 registers per SIMD lane hold
four wavefronts of up to 128, five of up to 96, and so on.  Kernels that wait for
memory lose speed with every wavefront they fall short of."""
import os
import re
import struct

import pytest

import paper_1010_5636_amd as ndq

msgpack = pytest.importorskip("msgpack")

NT_AMDGPU_METADATA = 32


def code_objects(blob):
    """The gfx950 code objects of every offload bundle in the library."""
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.start() + 24
        n, = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if name.endswith(b"gfx950") and size:
                yield blob[m.start() + off:m.start() + off + size]


def notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3a)
    for k in range(count):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + k * entsize)
        at, end = off, off + size
        while kind == 7 and at < end:   # SHT_NOTE
            namesz, descsz, ntype = struct.unpack_from("<III", elf, at)
            at += 12 + (namesz + 3) // 4 * 4
            yield ntype, elf[at:at + descsz]
            at += (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    path = os.path.join(os.path.dirname(ndq.__file__), "libndq.so")
    with open(path, "rb") as f:
        blob = f.read()
    out = {}
    for elf in code_objects(blob):
        for ntype, desc in notes(elf):
            if ntype == NT_AMDGPU_METADATA:
                for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                    out[k[".name"]] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
    assert out
    return out


def of(kernels, name, *args):
    """Registers and scratch of every instance of a kernel template with these first arguments."""
    tag = f"{len(name)}{name}I" + "".join(f"Li{a}E" for a in args)
    got = {k: v for k, v in kernels.items() if tag in k}
    assert got, tag
    return got


F16_LINKS = [(1, 18), (1, 12), (1, 8), (2, 18), (2, 12)]


@pytest.mark.parametrize("lp,recon", F16_LINKS)
@pytest.mark.parametrize("name", ["k_wilson_multi", "k_wilson_mrhs"])
def test_f16_fields_keep_four_wavefronts(kernels, name, lp, recon):
    for k, (registers, scratch) in of(kernels, name, 2, lp, recon).items():
        assert registers <= 128 and scratch == 0, (k, registers, scratch)


@pytest.mark.parametrize("nt", [0, 1])
def test_eight_fp64_reals_keep_three_wavefronts(kernels, nt):
    """The direction split without extra vectors."""
    got = [v for k, v in of(kernels, "k_wilson_dirsplit", 0, 0, 8).items() if f"Lb{nt}ELi0E" in k]
    assert len(got) == 1
    registers, scratch = got[0]
    assert registers <= 168 and scratch == 0
