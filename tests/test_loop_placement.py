"""Where the built library's code lies, for the loop whose speed depends on it (k_prefill.hpp, smallest tiles): its padding is sized
for what the compiler puts in front of it and would otherwise go out of step unseen."""
import os
import re
import subprocess

import pytest

from paper_2510_24273_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def _tool(name, *args):
    return subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True, text=True).stdout


def _innermost_matrix_loops(text):
    """(first address, bytes) of the innermost loops with matrix instructions in a function's disassembly."""
    code = [(int(m.group(2), 16), m.group(1).strip()) for m in re.finditer(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", text, re.M)]
    loops = []
    for at, ins in code:
        m = re.match(r"s_c?branch\S* (\d+)", ins)
        if m and int(m.group(1)) >= 1 << 15:   # backward: the offset counts words from the next instruction
            first = at + 4 + 4 * (int(m.group(1)) - (1 << 16))
            if any(first <= a < at and "mfma" in i for a, i in code):
                loops.append((first, at + 4 - first))
    return [x for x in loops if not any(y != x and x[0] <= y[0] and y[0] + y[1] <= x[0] + x[1] for y in loops)]


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="no LLVM tools")
@pytest.mark.parametrize("kernel", ["prefill_tile_kernelILi1ELi1E", "prefill_split_kernelILi4ELi1E", "prefill_split_kernelILi5ELi1E"])
def test_loop_of_the_smallest_prompt_tiles_starts_a_cache_line(kernel, tmp_path):
    if build.is_stale():
        build.build()
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    _tool("llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, build.LIB, os.devnull)
    _tool("clang-offload-bundler", "--unbundle", "--type=o", "--input=" + bundle, "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + code)
    names = [w for w in _tool("llvm-readelf", "--symbols", "--wide", code).split() if kernel in w and not w.endswith(".kd")]
    assert names
    loops = _innermost_matrix_loops(_tool("llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + names[0], code))
    small = [first for first, size in loops if size < 768]   # (eight matrix instructions: 612 to 636 bytes; the larger tiles' are longer)
    assert small and all(first % 64 == 0 for first in small), loops
