"""What the compiler cannot check in the kernel sources."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_inline_assembly_names_the_special_registers_it_writes():
    seen = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2403_17312_amd", "csrc", "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for asm in re.findall(r"\basm\s+volatile\s*\((.*?)\);", text, flags=re.S):
            code, _, operands = asm.partition(":")
            for reg in re.findall(r"\b(?:s_mov_b32|s_add_u32)\s+(m0)\b", code):
                seen += 1
                assert f'"{reg}"' in operands.rpartition(":")[2], f"{os.path.basename(path)}: {reg} is written and not named"
    assert seen


def test_a_wave_barrier_stands_between_fences():
    """The barrier of one wave orders no memory accesses for the compiler: where lanes exchange through LDS, fences have to."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2403_17312_amd", "csrc", "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__builtin_amdgcn_wave_barrier\(\);", text):
            seen += 1
            assert re.search(r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"[^;]*;\s*$', text[:m.start()]), os.path.basename(path)
            assert re.match(r'\s*__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"', text[m.end():]), os.path.basename(path)
    assert seen


def test_kernels_are_launched_in_one_way():
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2403_17312_amd", "csrc", "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        assert "<<<" not in text and "hipLaunchKernelGGL" not in text, os.path.basename(path)
        assert ("hipLaunchKernel(" in text) == path.endswith("swa_kernels.hpp"), os.path.basename(path)
