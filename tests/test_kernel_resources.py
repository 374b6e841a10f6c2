"""What the compiler made of the kernels, as the built library's own metadata says."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2511_15618_amd import binding

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


def _device_code(data: bytes) -> bytes:
    """The gfx950 code object inside the shared library (an ELF of machine AMDGPU = 224)."""
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:
            return data[at:]
        at = data.find(b"\x7fELF", at + 4)
    raise AssertionError("no device code in the library")


def _scratch(notes: str) -> dict:
    """Bytes of scratch memory per lane, by kernel."""
    return {name: int(size) for name, size in
            re.findall(r"\.name:\s+(_Z\w*k_\w+)\n(?:\s+\.(?!name)\w+:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", notes)}


def _notes(tmp_path) -> str:
    if not os.path.exists(binding.LIB_PATH):
        from paper_2511_15618_amd import build
        build.build()
    obj = tmp_path / "device.elf"
    obj.write_bytes(_device_code(open(binding.LIB_PATH, "rb").read()))
    return subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout


def _kernels(tmp_path) -> dict:
    return _scratch(_notes(tmp_path))


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_no_kernel_needs_scratch_memory(tmp_path):
    """Registers that do not fit go to memory, lane by lane: every kernel here is written to stay within its registers."""
    scratch = _kernels(tmp_path)
    assert len(scratch) > 100 and any("k_merge" in k for k in scratch) and any("k_verify_persist" in k for k in scratch)
    assert {k: n for k, n in scratch.items() if n} == {}


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_every_instance_of_the_single_launch_kernel_has_a_lockstep_case(tmp_path):
    """Row groups and width as the kernel's template parameters have them; a width without an instance of its own runs the general one."""
    from test_gpu_decode_kernels import CASES
    built = {tuple(map(int, m)) for k in _kernels(tmp_path) for m in re.findall(r"k_verify_persistILi(\d)ELi(\d+)E", k)}
    assert {(1, 0), (2, 0)} <= built
    run = set()
    for c in CASES:
        if c.name.startswith("one_launch"):
            sized = (2 if c.block_max > 16 else 1, c.d_model // 128 if c.ffn_mult == 4 else 0)
            run.add(sized if sized in built else (sized[0], 0))
    assert run == built


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_the_single_launch_kernel_stays_small(tmp_path):
    """One loop over the stages with one instance of each unit's code: 27 to 40 KB an instance and 82 to 180 scalars that do not fit their registers.  With code of its
    own for every stage of a block it was 56 to 88 KB and 173 to 308.  Two compute units hold 64 KB of instructions together."""
    spills = {m[0]: int(m[1]) for m in re.findall(r"\.name:\s+(_Z\w*k_verify_persist\w+)\n(?:\s+\.(?!name)\w+:.*\n)*?\s+\.sgpr_spill_count:\s+(\d+)", _notes(tmp_path))}
    symbols = subprocess.run([READELF, "--symbols", "--wide", str(tmp_path / "device.elf")], capture_output=True, text=True, check=True).stdout
    code = {f[7]: int(f[2], 0) for f in (line.split() for line in symbols.splitlines()) if len(f) > 7 and f[3] == "FUNC" and f[7] in spills}
    assert len(spills) == 14 and code.keys() == spills.keys()
    assert {k: n for k, n in code.items() if n > 50000} == {}
    assert {k: n for k, n in spills.items() if n > 190} == {}
