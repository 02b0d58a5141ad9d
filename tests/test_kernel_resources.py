"""Registers and scratch of the built kernels where a wave more or fewer per SIMD
was measured to matter: read from the metadata of the library's own code objects.
No GPU needed; skipped when the toolchain's readelf is absent."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled kernel name -> (vector registers, scratch bytes)."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not available")
    from paper_2009_03254_amd import _capi
    if not os.path.exists(_capi.LIB_PATH):
        from paper_2009_03254_amd import build
        build.build()
    with open(_capi.LIB_PATH, "rb") as fh:
        lib = fh.read()
    out, path = {}, str(tmp_path_factory.mktemp("co") / "k.elf")
    for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", lib):   # ELF64, OS ABI: HSA
        with open(path, "wb") as fh:
            fh.write(lib[m.start():])
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"^    \.name:\s+(\S+)", k, re.M).group(1)
            vgprs, scratch = (int(re.search(rf"\.{key}:\s+(\d+)", k).group(1))
                              for key in ("vgpr_count", "private_segment_fixed_size"))
            out[name] = (vgprs, scratch)
    assert out, "no code objects found"
    return out


@pytest.mark.parametrize("kernel,vgprs", [
    ("k_cullILb1ELi8E", 128),   # the queued cull: 4 waves per SIMD
])
def test_registers(kernels, kernel, vgprs):
    got = [v for k, v in kernels.items() if kernel in k]
    assert len(got) == 1, sorted(kernels)
    assert got[0][0] <= vgprs and got[0][1] == 0, got
