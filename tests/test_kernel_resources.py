"""Register use that the set-up kernels depend on, read from the metadata of the library's own
gfx950 code objects.  The local condensation keeps a row of [A | B | Mtilde] in registers; an
index into that row which is not a constant moves it to scratch memory (256x256 torus, p = 3:
8.8 ms instead of 3.2), without an error."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2004_09389_amd", "libhdg.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of the library's offload bundles (magic, entry count, then
    offset, size and target name of each entry)."""
    for m in re.finditer(MAGIC, data):
        base = m.start()
        (count,) = struct.unpack_from("<Q", data, base + len(MAGIC))
        at = base + len(MAGIC) + 8
        for _ in range(count):
            off, size, name = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + name].decode()
            at += 24 + name
            if "gfx950" in target and size:
                yield data[base + off:base + off + size]


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Scratch bytes per lane of every kernel, by mangled name."""
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("library or llvm-readelf not here")
    with open(LIB, "rb") as f:
        data = f.read()
    out = {}
    path = tmp_path_factory.mktemp("co") / "code.o"
    for obj in code_objects(data):
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.a", notes):   # an entry of amdhsa.kernels begins with its .agpr_count
            name = re.search(r"\n\s+\.name:\s+(\S+)", kernel)
            size = re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel)
            if name and size:
                out[name.group(1)] = int(size.group(1))
    return out


def test_local_condensation_stays_in_registers(scratch):
    kernels = {k: v for k, v in scratch.items() if "k_cell_condense" in k and "k_cell_condenseI" in k}
    assert len(kernels) == 6, sorted(kernels)   # p = 1..3, both fluxes
    assert all(v == 0 for v in kernels.values()), kernels
