"""Registers and scratch memory of the built kernels, from the code object's own metadata (no GPU).

The vector-ALU kernels hide memory latency with wavefronts, and a second body in a kernel (the right-hand strips) costs the first its registers: lines
below are what the wavefronts a SIMD were measured with (512 registers a SIMD lane, allocated in eights).
"""
import os
import re
import subprocess

import pytest

from paper_2010_15884_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("code")
    fat, obj = str(tmp / "fat"), str(tmp / "code.o")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", B.LIB_PATH, str(tmp / "unused")], check=True)
    data = open(fat, "rb").read()
    found = {}
    # one bundle per translation unit
    starts = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)]
    for a, b in zip(starts, starts[1:] + [len(data)]):
        open(fat, "wb").write(data[a:b])
        subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={fat}", f"--output={obj}",
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", obj], check=True, capture_output=True, text=True).stdout
        for entry in notes.split("  - .agpr_count")[1:]:
            field = lambda n: re.search(rf"\.{n}:\s+(\S+)", entry).group(1)
            found[field("name")] = {n: int(field(n)) for n in ("vgpr_count", "sgpr_count", "sgpr_spill_count", "private_segment_fixed_size")}
            sizes = re.search(r"\.args:(.*?)\.group_segment", entry, re.S).group(1)
            found[field("name")]["first_argument"] = next((int(v) for o, v in re.findall(r"\.offset:\s+(\d+)\s+\.size:\s+(\d+)", sizes) if o == "0"), 0)
    assert len(found) > 200
    return found


def test_no_kernel_uses_scratch_memory(kernels):
    assert not [n for n, r in kernels.items() if r["private_segment_fixed_size"]]


@pytest.mark.parametrize("k,most", [(8, 80), (9, 72), (10, 88), (11, 90)])
def test_bfs_strips_keep_their_wavefronts(kernels, k, most):
    mine = [r["vgpr_count"] for n, r in kernels.items() if f"conv2d_bfs_kernelILi{k}E" in n]
    assert mine and max(mine) <= most


@pytest.mark.parametrize("k,vector,scalar", [(2, 22, 43), (3, 28, 50), (4, 38, 62), (5, 51, 65), (6, 68, 92), (7, 89, 106)])
def test_bfs_blocks_on_whole_quads_keep_their_registers(kernels, k, vector, scalar):
    """kNarrow (2), the kernel for widths that are multiples of four: what it had before clamped loads came to the others."""
    mine = [r for n, r in kernels.items() if f"conv2d_bfs_block_kernelILi{k}E" in n and "StripKindE2" in n]
    assert len(mine) == 1 and mine[0]["vgpr_count"] <= vector and mine[0]["sgpr_count"] <= scalar


def test_arguments_behind_the_taps_begin_a_block_of_their_own(kernels):
    taps = {n: r["first_argument"] for n, r in kernels.items() if "TapsOf" in n}
    assert len(taps) > 100
    assert not {n: b for n, b in taps.items() if b < 256 or b > 1024}


@pytest.mark.parametrize("rows", [2, 3, 4])
def test_stride2_pairs_keep_their_taps_in_scalar_registers(kernels, rows):
    """From 8 columns on (up to 64 vector registers leave eight wavefronts a SIMD; four rows of nine columns do not fit the scalar ones, and ten go to lanes of a vector register)."""
    mine = {n: r for n, r in kernels.items() for k in range(8, 16) if f"conv2d_fbs_stride2_pair_kernelILi{k}ELi{rows}E" in n}
    assert len(mine) == {2: 8, 3: 6, 4: 4}[rows]                # three rows: all but 10 and 11 columns; four: up to 11
    assert not {n: r for n, r in mine.items() if r["vgpr_count"] > 48 or r["sgpr_spill_count"] > 12}


@pytest.mark.parametrize("k,rows", [(k, r) for k in range(12, 16) for r in (1, 2, 3, 4)])
def test_fbs_strips_keep_their_taps_in_scalar_registers(kernels, k, rows):
    mine = [r for n, r in kernels.items() if f"conv2d_fbs_strip_kernelILi{k}ELi{rows}E" in n]
    assert len(mine) == 1 and mine[0]["vgpr_count"] <= 56 and mine[0]["sgpr_spill_count"] == 0
