"""What the compiler made of the kernels, read from the library's own code
objects (built here, for gfx950)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1206_3229_amd import vlasov as V

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no LLVM binary tools")
    V.load()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(V.LIB_PATH, d)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, cwd=d, capture_output=True)
    found = sorted(str(p) for p in d.iterdir() if "gfx950" in p.name)
    assert found
    return found


def _kernels(code_object):
    """Kernel symbols of a code object and their metadata, as text."""
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object], check=True,
                           capture_output=True, text=True).stdout
    for entry in notes.split("  - .agpr_count:")[1:]:
        yield re.search(r"\.symbol:\s+'?(\S+?)\.kd", entry).group(1), entry


def test_half_drifts_of_long_lines_load_16_bytes(code_objects):
    """Both storages, boundaries, one and two half drifts, written through and back."""
    seen = set()
    for co in code_objects:
        for name, _ in _kernels(co):
            m = re.match(r"_ZN2vkL7k_driftI([fd])Li([01])ELi([12])ELb([01])ELb1EE", name)
            if m and m.groups() not in seen:
                seen.add(m.groups())
                text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", f"--disassemble-symbols={name}", co],
                                      check=True, capture_output=True, text=True).stdout
                loads = re.findall(r"global_load_dword\S*", text)
                assert loads.count("global_load_dwordx4") >= 8, (name, loads)
    assert len(seen) == 16


def test_batch_kernels_do_not_spill(code_objects):
    """The batched drift and fused kernel hold eight tile kinds in one loop over the work items."""
    seen = set()
    for co in code_objects:
        for name, meta in _kernels(co):
            m = re.match(r"_ZN2vkL(?:8kb_drift|13kb_kick_drift)I([fd])", name)
            if m:
                seen.add(name)
                for key in (".vgpr_spill_count", ".private_segment_fixed_size"):
                    assert re.search(re.escape(key) + r":\s+0\b", meta), (name, key)
    assert len(seen) == 4
