"""What the compiler makes of the kernels where a source that reads well can lose what it is written for: the AMD assembly
of this repository's own sources."""
import os
import re
import subprocess

from paper_2009_06693_amd import build


def _kernels(tmp_path, source, pattern):
    """(name, instructions) of the kernels whose mangled name matches."""
    asm = tmp_path / (source + ".s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(asm)],
                   check=True, capture_output=True)
    for name, body in re.findall(r"\n(_ZN\w*" + pattern + r"\w*):[^\n]*\n(.*?)\.Lfunc_end", asm.read_text(), re.S):
        code = [line.split(";")[0].strip() for line in body.splitlines()]
        yield name, [line for line in code if line]


def test_packed_columns_are_loaded_side_by_side(tmp_path):
    """The four loads of a lane in the last hop of k-hop are waited for together.  Where a branch held the load and the taking
    of the bits, each load was waited for before the next was issued (300 K vertices of 3 M, [8,8,4], 1,202 us, 1,158 side
    by side)."""
    kernels = list(_kernels(tmp_path, "nd_khop.hip", r"khop_fused_kernelILi\dELi\dELb\dELb1E"))
    assert len(kernels) == 16
    for name, code in kernels:
        taken = [i for i, line in enumerate(code) if re.match(r"v_bfe_u32 v\d+, v\d+, v\d+, s\d+", line)]
        assert len(taken) == 4, name
        assert sum("vmcnt(0)" in code[i - 1] for i in taken) <= 1, name
