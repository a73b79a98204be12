"""The code generated for the small solve's hand-over of chunk sums between workgroups."""

import os
import re
import subprocess

from paper_2608_21607_amd import build


def test_chunk_sums_are_stored_before_they_are_counted(tmp_path):
    """A workgroup's partial is read by whichever workgroup counts last, perhaps behind another L2.
    The thread that writes the L2 back and counts waits for its own wave's stores only, so every
    wave has to have waited for its own before the barrier that thread passes."""
    out = tmp_path / "chol.s"
    subprocess.run([build.hipcc(), *build.HIPFLAGS, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "chol.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    kernels = {}
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        if m := re.match(r"(_ZN3nmd1\d(solve_small|solve_sparse)_kernel\w+):", line):
            code = kernels.setdefault(m.group(1), [])
        elif kernels and line.startswith((".Lfunc_end", ".section")):
            code = []
        elif kernels and line:
            code.append(line)
    assert len(kernels) == 8  # both launches at each rank
    for name, code in kernels.items():
        counts = [i for i, c in enumerate(code) if c.startswith("global_atomic_add")]
        assert len(counts) == 1, name
        barrier = max(i for i in range(counts[0]) if code[i].startswith("s_barrier"))
        store = max(i for i in range(barrier) if code[i].startswith("global_store"))
        waits = [c for c in code[store:barrier] if c.startswith("s_waitcnt") and "vmcnt(0)" in c]
        assert waits, f"{name}: {code[store:barrier + 1]}"
