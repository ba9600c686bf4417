"""What the built kernels use, from the notes of libwd's own code objects (no GPU)."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    """Kernel name -> its notes (numbers)."""
    from paper_2108_13976_amd import build

    scratch = tmp_path_factory.mktemp("code_objects")
    os.symlink(build.LIBRARY, scratch / "libwd.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "libwd.so"], cwd=scratch, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for name in os.listdir(scratch):
        if not name.endswith("gfx950"):
            continue
        text = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", name], cwd=scratch, check=True, stdout=subprocess.PIPE, text=True).stdout
        for part in text.split("- .agpr_count")[1:]:
            kernel = re.search(r"\.name:\s+(\S+)", part[part.index(".max_flat_workgroup_size"):]).group(1)
            found[kernel] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s*$", part, flags=re.M)}
    return found


def test_no_registers_in_scratch_memory(notes):
    """The kernels whose time is a chain of instructions keep every variant's state in registers."""
    served = [k for k in notes if re.search("quad_env_kernel|crew_env_kernel", k)]
    assert len(served) == 6 + 21, sorted(served)
    for k in served:
        assert notes[k]["private_segment_fixed_size"] == 0 and notes[k]["vgpr_spill_count"] == 0, (k, notes[k])
