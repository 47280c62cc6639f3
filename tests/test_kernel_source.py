"""Rules for the kernels' source that no run can show to be kept: what breaks them fails rarely, or hangs."""
import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04450_amd", "csrc")


def sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(path) as f:
            yield os.path.basename(path), re.sub(r"//[^\n]*|/\*.*?\*/", "", f.read(), flags=re.S)


def test_no_block_waits_for_another_one():
    # blocks of an ordinary launch need not all be resident: a loop on a word that other blocks set may never end
    for name, code in sources():
        assert "s_sleep" not in code, name
        assert not re.search(r"\b(while|for)\s*\([^{};]*atomic", code), name
        assert not re.search(r"cooperative|grid\.sync", code), name


def test_assembly_that_needs_m0_sets_it_and_says_so():
    # the compiler may use m0 between any two statements: one that copies to LDS sets it itself, and names it as changed
    found = 0
    for name, code in sources():
        for asm in re.findall(r"\basm\s+volatile\s*\((.*?)\)\s*;", code, flags=re.S):
            if "m0" not in asm and "load_lds" not in asm:
                continue
            found += 1
            text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', asm.split("::")[0]))
            assert re.match(r"s_mov_b32 m0, %0\\n\\ts_nop \d\\n\\tglobal_load_lds", text), (name, asm)
            assert re.search(r':\s*[^:]*"m0"\s*$', asm), (name, asm)
    assert found


@pytest.mark.parametrize("name", ["emb_kernels.hip", "hstu_kernels.hip", "hstu_fp32.hip"])
def test_scalar_registers_leave_room_for_eight_wavefronts(name, tmp_path):
    # 800 scalar registers per SIMD in sixteens, sixteen more per wavefront than the compiler counts: a kernel whose vector
    # registers allow eight wavefronts (64 each) keeps them only with 80 scalar ones
    asm = tmp_path / "kernels.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-w", "--cuda-device-only", "-S", os.path.join(CSRC, name), "-o", str(asm)], check=True)
    found = 0
    for entry in re.split(r"\n  - \.agpr_count:", asm.read_text())[1:]:
        field = lambda key: re.search(r"\.%s:\s+(\S+)" % key, entry).group(1)
        vector = int(entry.split()[0]) + int(field("vgpr_count"))
        found += 1
        if vector <= 64:
            assert int(field("sgpr_count")) <= 80, field("name")
    assert found >= 5


def test_settling_whole_sets_keeps_its_registers(tmp_path):
    # it runs behind every lookup of up to 32 768 ids, also where nothing was missing: no scratch memory, in any of its forms
    asm = tmp_path / "kernels.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-w", "--cuda-device-only", "-S", os.path.join(CSRC, "emb_kernels.hip"), "-o", str(asm)], check=True)
    scratch = {}
    for entry in re.split(r"\n  - \.agpr_count:", asm.read_text())[1:]:
        name = re.search(r"\.name:\s+(\S+)", entry).group(1)
        if "miss_settle_sets" in name:
            scratch[name] = re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry).group(1)
    assert scratch and set(scratch.values()) == {"0"}, scratch


def test_joined_halves_fit_the_blocks_per_cu_that_the_rule_counts(tmp_path):
    # join_slices brings no more blocks than the chip holds at once: two per CU, one at d = 512, a wavefront per SIMD each, of 512
    # registers per SIMD and lane and 160 KB of LDS per CU
    asm = tmp_path / "kernels.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-w", "--cuda-device-only", "-S", os.path.join(CSRC, "hstu_kernels.hip"), "-o", str(asm)], check=True)
    found = 0
    for entry in re.split(r"\n  - \.agpr_count:", asm.read_text())[1:]:
        field = lambda key: re.search(r"\.%s:\s+(\S+)" % key, entry).group(1)
        width = re.search(r"layer_(?:join|first)ILi(\d+)E", field("name"))
        if not width:
            continue
        found += 1
        per_cu = 2 if int(width.group(1)) <= 256 else 1
        registers = -(-int(field("vgpr_count")) // 8) * 8  # accumulation registers are counted in
        assert registers * per_cu <= 512, (field("name"), registers)
        assert int(field("group_segment_fixed_size")) * per_cu <= 160 * 1024, field("name")
        assert field("private_segment_fixed_size") == "0", field("name")
    assert found == 16  # four widths: both halves, either alone, and the one that begins a step
