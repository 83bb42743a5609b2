"""Properties of the built kernels that the sources cannot state, read from the library's own gfx950 code objects."""
import os
import re
import subprocess

import pytest

from paper_2511_11641_amd import build as bld

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The device code objects inside the library, one file per translation unit."""
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no LLVM tools")
    if not os.path.exists(bld.LIB):
        bld.build(verbose=False)
    d = tmp_path_factory.mktemp("co")
    os.symlink(bld.LIB, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    files = sorted(str(d / f) for f in os.listdir(d) if "gfx950" in f)
    assert files
    return files


def test_no_scratch_memory(code_objects):
    """Every kernel of a pass keeps its values in registers (spills would travel beside the direct loads of the main loops)."""
    scratch = {}
    for f in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f], check=True, capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, flags=re.S):
            scratch[name] = int(size)
    assert len(scratch) > 100
    assert {n: s for n, s in scratch.items() if s and "mfma_probe" not in n} == {}
