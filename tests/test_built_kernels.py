"""What the built library holds, read from its own symbols (no GPU)."""
import collections
import os
import re
import struct
import subprocess

from paper_1901_03040_amd import binding, build


def test_every_kernel_is_built_once():
    """Each unit's copy of a kernel has its own host stub, local to the unit: two of one name are two copies of the device code."""
    binding.lib()
    table = subprocess.run(["nm", build.LIB], capture_output=True, text=True, check=True).stdout
    stubs = collections.Counter(line.split()[-1] for line in table.splitlines() if "__device_stub__" in line)
    assert any("k_round_fused" in n for n in stubs) and any("k_quantize_pack_fast" in n for n in stubs)
    assert [n for n, copies in stubs.items() if copies > 1] == []


READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def kernel_notes(tmp_path):
    """{kernel symbol: its notes' plain numbers} of all gfx950 code objects in the library."""
    with open(build.LIB, "rb") as f:
        lib = f.read()
    out = {}
    for bundle in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", lib):
        at = bundle.end()
        count, = struct.unpack_from("<Q", lib, at)
        at += 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", lib, at)
            triple = lib[at + 24:at + 24 + name].decode()
            at += 24 + name
            if not triple.endswith("gfx950") or size == 0:
                continue
            path = tmp_path / f"{bundle.start()}.o"
            path.write_bytes(lib[bundle.start() + offset:bundle.start() + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for kernel in re.split(r"\n  - (?=\.)", notes)[1:]:
                symbol = re.search(r"\.symbol:\s*'?(\S+?)\.kd'?\s", kernel)
                if symbol:
                    out[symbol.group(1)] = {k: int(v) for k, v in re.findall(r"\n    \.(\w+):\s*(\d+)\b", "\n    " + kernel)}
    return out


def test_two_workgroups_of_sixteen_waves_fit_a_cu(tmp_path):
    """Where the vector registers allow two (512 per lane and SIMD, eight waves), the scalar ones do too: 800 per SIMD, handed
    out in steps of 16, 16 of them per wave to the trap handler, which the compiler does not count."""
    kernels = {n: k for n, k in kernel_notes(tmp_path).items()
               if "k_quantize_pack" in n and k["max_flat_workgroup_size"] == 1024 and k["vgpr_count"] <= 64}
    assert any("k_quantize_pack_bucket" in n for n in kernels) and any("k_quantize_pack_fast" in n for n in kernels)
    assert {n: k["sgpr_count"] for n, k in kernels.items() if k["sgpr_count"] > 80} == {}


def host_values(tmp_path, body):
    """Output of a program that sees the library's host-side rules (no HIP call is made)."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include "qesgd_internal.h"\n#include <cstdio>\nusing namespace qesgd;\nint main() {\n' + body + "\nreturn 0; }\n")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-Wno-deprecated-declarations", "-I/opt/rocm/include",
                    f"-I{os.path.join(build.ROOT, 'include')}", f"-I{build.CSRC}", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout


def test_streaming_kernels_hold_six_waves_per_simd(tmp_path):
    """The LDS that a streaming launch asks for, with what the built kernel has itself, leaves a CU 24 waves for workgroups of 2, 4
    and 8 waves (buckets of 8192 among them); those of 16 ask for none."""
    out = host_values(tmp_path, 'for (unsigned w : {2u, 4u, 8u, 16u}) std::printf("%u %u\\n", w, six_wave_lds(w, 0));')
    ask = {int(w): int(b) for w, b in (line.split() for line in out.splitlines())}
    assert ask.pop(16) == 0
    seen = set()
    for name, k in kernel_notes(tmp_path).items():
        if not re.search("k_quantize_pack_fast|k_tile_partials_fast|k_quantize_pack_pre_fast", name):
            continue
        waves = k["max_flat_workgroup_size"] // 64
        if waves == 16:
            continue
        seen.add(waves)
        assert k["group_segment_fixed_size"] < ask[waves]
        assert 160 * 1024 // ask[waves] * waves == 24 and ask[waves] % 1280 == 0, name
        assert k["vgpr_count"] <= 80, name                   # otherwise the registers allow fewer than six anyway
    assert seen == {2, 4, 8}
