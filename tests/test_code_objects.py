"""Register spills of the moment-form adjoint kernels, from the code objects' own metadata (no GPU)."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2607_18074_amd import _lib

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _scratch(path):
    notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
    kernels = re.findall(r"\.name: +(\S+).*?\.private_segment_fixed_size: (\d+)", notes, re.S)
    return {n: int(b) for n, b in kernels if n.startswith("sobek_adj_")}


@pytest.mark.skipif(not os.path.exists(READELF), reason="ROCm llvm-readelf not found")
def test_many_narrow_groups_do_not_spill():
    """16-channel blocks would pack 128x0e+64x1o+64x2e+64x3o into the fewest steps (88, in eleven groups written out
    one after the other: 1,244 bytes of spilled registers a lane, 1.5 to 3.5 times the per-edge kernels' time)."""
    sig = ("128x0e+64x1o+64x2e+64x3o", 3, "128x0e+64x1o+64x2e+64x3o", 16)
    cache = os.environ.get("SOBEK_JIT_CACHE") or os.path.join(os.path.dirname(os.path.abspath(_lib.__file__)), "_jitcache")
    os.makedirs(cache, exist_ok=True)

    def objects():
        return {f: os.path.getmtime(os.path.join(cache, f)) for f in os.listdir(cache) if f.endswith(".co")}

    before = objects()
    _lib.jit_compile(*sig)   # a hit renews the object's time
    scratch = {}
    for f, t in objects().items():
        if before.get(f) != t:
            scratch.update(_scratch(os.path.join(cache, f)))
    assert set(scratch) == {"sobek_adj_E", "sobek_adj_dE"}
    assert max(scratch.values()) <= 512, scratch
