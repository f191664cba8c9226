"""What the built library holds, read from its own symbols (no GPU)."""
import collections
import subprocess

from paper_1901_03040_amd import binding, build


def test_every_kernel_is_built_once():
    """Each unit's copy of a kernel has its own host stub, local to the unit: two of one name are two copies of the device code."""
    binding.lib()
    table = subprocess.run(["nm", build.LIB], capture_output=True, text=True, check=True).stdout
    stubs = collections.Counter(line.split()[-1] for line in table.splitlines() if "__device_stub__" in line)
    assert any("k_round_fused" in n for n in stubs) and any("k_quantize_pack_fast" in n for n in stubs)
    assert [n for n, copies in stubs.items() if copies > 1] == []
