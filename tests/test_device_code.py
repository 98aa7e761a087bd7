"""What the compiler made of load hints that nothing else would show: built for gfx950 from the kernels' header, no device."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_06069_amd", "csrc")
SOURCE = """#include "ob_kernels.h"
using namespace obk;
#define PASS(KEEP) template __global__ void obk::k_ratios_pass<1, false, false, KEEP>( \\
    RatioArgs, float*, int64_t, int, LayerTab, const int*, const int*, const int*);
PASS(false)
PASS(true)
"""


def test_second_reads_are_kept_only_where_asked_for(tmp_path):
    """The ratio pass loads m, v_frozen and v_fresh past the caches, or v_frozen through them: one hint less."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    src, asm = tmp_path / "pass.hip", tmp_path / "pass.s"
    src.write_text(SOURCE)
    subprocess.run([hipcc, "-O3", "--offload-arch=gfx950", "--offload-device-only", "-S", "-std=c++17", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    text, hints = asm.read_text(), []
    for keep in "01":
        body = re.search(r"^_ZN3obk13k_ratios_passILi1ELb0ELb0ELb%s\w*:[^\n]*$(.*?)s_endpgm" % keep, text, re.S | re.M).group(1)
        hints.append(len(re.findall(r"global_load_dwordx4 .* nt$", body, re.M)))
    assert hints == [3, 2], hints
