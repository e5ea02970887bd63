"""The counted waits for copies under way: the counter has six bits, and a count beyond them would wait for others than meant; it does not compile."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_09849_amd", "csrc")
WAIT = """#include <hip/hip_runtime.h>
#include "internal.hpp"
#include "regconv3.hpp"
__global__ void wait() { __builtin_amdgcn_s_waitcnt(hts::wait_imm<%d>()); }
"""


@pytest.mark.parametrize("count, compiles", [(0, True), (63, True), (64, False), (-1, False)])
def test_counts_beyond_the_counter_do_not_compile(tmp_path, count, compiles):
    source = tmp_path / "wait.hip"
    source.write_text(WAIT % count)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "-I", CSRC, str(source)], capture_output=True, text=True)
    assert (r.returncode == 0) == compiles, r.stderr
    assert compiles or "vmcnt has six bits" in r.stderr
