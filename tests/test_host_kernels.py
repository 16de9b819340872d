"""Registers of the render kernels, as the compiler noted them in the library built from this tree, and the compiler's warnings.

Eight wavefronts share a SIMD's 800 scalar registers, in steps of 16 and with 16 more for each than its kernel names: 80.
The kernels for whole frames rely on it (four workgroups of 512 threads, or two of 1024, on a compute unit), and a kernel
that needs more parks them in lanes of vector registers, an instruction for every use."""
import os
import re
import struct
import subprocess

import pytest

from paper_2502_00021_amd import build, pxr


def _code_objects(image):
    """The gfx950 ELF images in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(magic, image):
        at = m.start()
        n, = struct.unpack_from("<Q", image, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", image, p)
            name = image[p + 24:p + 24 + id_len]
            p += 24 + id_len
            if b"gfx950" in name and size:
                yield image[at + offset:at + offset + size]


def _notes(elf):
    """The AMDGPU metadata notes (type 32) of one code object."""
    sh_off, = struct.unpack_from("<Q", elf, 0x28)
    sh_size, sh_num = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(sh_num):
        sh_type, = struct.unpack_from("<I", elf, sh_off + k * sh_size + 4)
        offset, size = struct.unpack_from("<QQ", elf, sh_off + k * sh_size + 24)
        p = offset
        while sh_type == 7 and p < offset + size:
            name_len, desc_len, kind = struct.unpack_from("<III", elf, p)
            p += 12 + (name_len + 3) // 4 * 4
            if kind == 32:
                yield elf[p:p + desc_len]
            p += (desc_len + 3) // 4 * 4


def _render_kernels():
    msgpack = pytest.importorskip("msgpack")
    pxr.lib()  # (built if it is not)
    image = open(pxr.lib()._name, "rb").read()
    kernels = {}
    for elf in _code_objects(image):
        for note in _notes(elf):
            for k in msgpack.unpackb(note)["amdhsa.kernels"]:
                m = re.search(r"render_kernelILi(\d+)ELb([01])ELb([01])ELb([01])ELb([01])E", k[".name"])
                if m:
                    threads, ragged, windowed, video, posed = (int(g) for g in m.groups())
                    kernels[threads, ragged, windowed, video, posed] = k
    return kernels


def test_registers_of_the_render_kernels():
    kernels = _render_kernels()
    assert {k[:4] for k in kernels if not k[4]} == {(t, r, w, v) for t in (256, 512, 768, 1024) for r in (0, 1) for w in (0, 1) for v in (0, 1)}
    assert {k[:4] for k in kernels if k[4]} == {k[:4] for k in kernels if not k[2] or k[0] >= 768}
    for (threads, ragged, windowed, video, posed), k in kernels.items():
        where = dict(threads=threads, ragged=ragged, windowed=windowed, video=video, posed=posed)
        parked = k[".sgpr_spill_count"]
        if not windowed:
            assert k[".sgpr_count"] <= 80 and k[".vgpr_count"] <= 64, where
            # (by value where that is the faster form in spite of it: the largest workgroups without a clip)
            assert parked <= (6 if threads == 1024 and not video and not posed else 0), (where, parked)
            assert k[".private_segment_fixed_size"] == 0, where
        else:
            assert parked <= 24, (where, parked)


@pytest.mark.parametrize("source", build.SOURCES)
def test_sources_compile_without_warnings(source):
    """With the library's own flags, device pass and host pass."""
    flags = [f for f in build.HIPFLAGS if f != "-shared"]
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    include = ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC]
    r = subprocess.run([hipcc, *flags, "-fsyntax-only", "-Wno-unused-command-line-argument", *include, os.path.join(build.CSRC, source)],
                       stderr=subprocess.PIPE, text=True, check=True)
    assert "warning:" not in r.stderr, r.stderr[:2000]
