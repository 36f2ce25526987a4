"""Register allocation of the built kernels, read from the metadata in the library's code objects."""
import os
import re
import struct
import subprocess

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2504_07042_amd", "libaxhosfem.so")


def kernel_metadata(path):
    """{demangled name: metadata} of every kernel in the AMDGPU code objects embedded in `path`."""
    import msgpack
    data = open(path, "rb").read()
    found = []
    for m in re.finditer(b"\x7fELF", data):
        e = m.start()
        if struct.unpack_from("<H", data, e + 18)[0] != 224:   # EM_AMDGPU
            continue
        phoff, = struct.unpack_from("<Q", data, e + 32)
        phsize, phnum = struct.unpack_from("<HH", data, e + 54)
        for p in range(phnum):
            ph = e + phoff + p * phsize
            kind, = struct.unpack_from("<I", data, ph)
            off, = struct.unpack_from("<Q", data, ph + 8)
            size, = struct.unpack_from("<Q", data, ph + 32)
            if kind != 4:   # PT_NOTE
                continue
            q, end = e + off, e + off + size
            while q + 12 <= end:
                ns, ds, nt = struct.unpack_from("<III", data, q)
                desc = q + 12 + (ns + 3) // 4 * 4
                if nt == 32:   # NT_AMDGPU_METADATA
                    found += msgpack.unpackb(data[desc:desc + ds])["amdhsa.kernels"]
                q = desc + (ds + 3) // 4 * 4
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    return {n.replace("void ", "").replace("ax::", "").split("(")[0]: k for n, k in zip(names, found)}


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        from paper_2504_07042_amd import build
        build.build()
    ks = kernel_metadata(LIB)
    assert len(ks) > 500
    return ks


def test_cg_vector_kernels_do_not_spill(kernels):
    """They run at eight waves per SIMD, 64 registers."""
    names = [n for n in kernels if re.match(r"(qt_dot|update_dot|cg_dir)_kernel<", n)]
    assert len(names) == 11
    for n in names:
        k = kernels[n]
        assert (k[".vgpr_count"] <= 64, k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) == (True, 0, 0), (n, k)


def test_tile_kernels_spill_little(kernels):
    """The tile kernels in their default shape, single- and multi-column forms: no register spilled up
    to N1 = 9; above, at most 20 of 168 where one wave per SIMD fewer measured no faster."""
    default = {2: 16, 3: 7, 4: 4, 5: 5, 6: 7, 7: 5, 8: 1, 9: 3, 10: 3, 11: 2}   # elements per work-group
    seen = 0
    for n, k in kernels.items():
        m = re.match(r"ax_local_kernel<(\d+), \d, true, 0, (\d+), (true|false), (double|float)>", n)
        if m and int(m[2]) == default.get(int(m[1]), 1):
            seen += 1
            assert k[".vgpr_spill_count"] <= (0 if int(m[1]) <= 9 else 20), (n, k[".vgpr_spill_count"])
    assert seen == 15 * 2 * (2 + 3 * 2)
