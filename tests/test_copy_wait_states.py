"""The LDS copies that are written as inline assembly: the compiler keeps no distances to what is inside, so no vector instruction
may write a copy's scalars within the five wait states before it, and m0 has to be written one ahead.  Read from the built library."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNELS = ("wgrad_dma_kernel", "regconv_kernel", "DmaJob")


def scalars(operand):
    """Numbers of the scalar registers that an operand names."""
    one, many = re.fullmatch(r"s(\d+)", operand), re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return {int(one.group(1))} if one else set(range(int(many.group(1)), int(many.group(2)) + 1)) if many else set()


def operands(line):
    return [x.strip() for x in re.split(r",|\s(?=offen|offset|lds)", line.split(None, 1)[1])] if " " in line else []


def too_close(body):
    """The copies of a kernel's instructions that follow a vector instruction's write of one of their scalars too closely (distances
    along the text: a branch that is taken takes longer)."""
    bad = []
    for i, line in enumerate(body):
        if not (line.startswith("buffer_load") and re.search(r"\blds\b", line)):
            continue
        used = set().union(*(scalars(x) for x in operands(line)))
        states, j = 0, i - 1
        while states < 5 and j >= 0:
            if body[j].startswith("v_") and operands(body[j]) and scalars(operands(body[j])[0]) & used:
                bad.append(body[j:i + 1])
            nop = re.match(r"s_nop (\d+)", body[j])
            states += int(nop.group(1)) + 1 if nop else 1
            j -= 1
        if "m0" in body[i - 1]:
            bad.append(body[i - 1:i + 1])
    return bad


def test_finds_what_is_too_close():
    copy = "buffer_load_dwordx4 v4, s[12:15], s10 offen lds"
    for before, found in ((["v_readfirstlane_b32 s13, v2", "s_mov_b32 m0, s9", "s_nop 0"], True), (["v_readlane_b32 s10, v2, 3", "s_nop 2", "s_mov_b32 m0, s9", "s_nop 0"], False),
                          (["v_readlane_b32 s10, v2, 3", "s_nop 1", "s_mov_b32 m0, s9", "s_nop 0"], True), (["v_readlane_b32 s11, v2, 3", "s_mov_b32 m0, s9", "s_nop 0"], False),
                          (["s_add_i32 s10, s9, 4", "s_mov_b32 m0, s9", "s_nop 0"], False), (["s_nop 4", "s_mov_b32 m0, s9"], True)):
        assert bool(too_close(before + [copy])) == found, before


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")
def test_copies_keep_their_distances(tmp_path):
    from paper_2012_09849_amd import binding, build
    binding.load_library()
    lib = shutil.copy(build.LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    seen = set()
    for code in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(code)], check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^\s*$|\Z)", text, flags=re.S | re.M):
            kinds = [k for k in KERNELS if k in name]
            if kinds:
                lines = [line.split("//")[0].strip() for line in body.splitlines()]
                assert any(line.startswith("buffer_load") and line.endswith(" lds") for line in lines), name
                assert not too_close(lines), name
                seen.update(kinds)
    assert seen == set(KERNELS)
