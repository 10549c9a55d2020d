"""What the compiler made of the kernels, read from the built library: code properties that no result shows."""
import os
import re
import struct
import subprocess

import pytest

from paper_2511_05534_amd import build

LLVM = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="no LLVM tools")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code object of every source file, as files."""
    from paper_2511_05534_amd import binding
    binding.load()
    data = open(build.library_path(), "rb").read()
    files, at = [], data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if data[entry + 24:entry + 24 + name].endswith(b"gfx950"):
                files.append(tmp_path_factory.mktemp("code") / "object.elf")
                files[-1].write_bytes(data[at + offset:at + offset + size])
            entry += 24 + name
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    assert files
    return files


def _tool(name, *args):
    return subprocess.run([f"{LLVM}/{name}", *args], capture_output=True, text=True, check=True).stdout


def test_partial_sums_arrive_before_their_wave_counts_itself(code_objects):
    """Merge of a slot by several waves: between the stores of a wave's sums, which go past the caches of one XCD, and the count of the waves that
    are done stands a wait for all of its stores."""
    seen = 0
    for path in code_objects:
        if "merge_tasks_kernel" not in _tool("llvm-readelf", "--notes", path):
            continue
        for body in re.split(r"^[0-9a-f]+ <", _tool("llvm-objdump", "-d", "--no-show-raw-insn", path), flags=re.M):
            if "merge_tasks_kernel" not in body.split("\n", 1)[0]:
                continue
            code = [line.split("//")[0].split() for line in body.split("\n")[1:]]
            code = [c for c in code if c]
            count, = [i for i, c in enumerate(code) if c[0].startswith("global_atomic_add")]
            stores = [i for i, c in enumerate(code[:count]) if c[0].startswith("global_store") and c[-1] == "sc1"]
            waits = [i for i, c in enumerate(code[:count]) if c[0] == "s_waitcnt" and "vmcnt(0)" in " ".join(c)]
            assert stores and waits and stores[-1] < waits[-1], body.split("\n", 1)[0]
            assert not any("store" in c[0] for c in code[waits[-1]:count])
            loads = [c for c in code[count:] if c[0].startswith("global_load_dwordx2")]
            assert loads and all(c[-1] == "sc1" for c in loads), loads  # the other waves' sums
            seen += 1
    assert seen == 16, seen


# kernels (mangled), registers of a lane at the most, of bytes of scratch a lane none: what the workgroups that share a compute unit rest on
REGISTERS = {
    "unit_plan_kernelILb1E(Li[0-9]+E){2}Li1E": 80,  # bf16, one key tile a wave: six waves per SIMD
    "unit_plan_kernelILb0ELi64ELi[0-9]+ELi1E.*OperandE0E": 80,  # fp32 rows that are not split into terms: the same
    "unit_plan_kernelILb0ELi128ELi[0-9]+ELi1E.*OperandE0E": 128,  # four waves per SIMD
    "unit_m(atch|erge)_kernelILb0ELi64ELi256E": 128,  # fp32 match and merge, four workgroups of four waves
}


@pytest.mark.parametrize("kernel", list(REGISTERS))
def test_registers_leave_room_for_the_workgroups(code_objects, kernel):
    seen = 0
    for path in code_objects:
        for entry in _tool("llvm-readelf", "--notes", path).split("- .agpr_count:")[1:]:
            value = lambda key: re.search(rf"\.{key}: +(\S+)", entry).group(1)
            if re.search(kernel, value("name")):
                assert int(value("vgpr_count")) <= REGISTERS[kernel], entry  # (accumulation registers among them)
                assert int(value("private_segment_fixed_size")) == 0, value("name")
                seen += 1
    assert seen
