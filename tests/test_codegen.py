"""What the compiler makes of kernels that are bound by the width of their loads: the sources are
compiled to gfx950 assembly and the loads are counted."""
import os
import re
import subprocess

import pytest

from paper_2511_05589_amd import build


def _assembly(source, tmp_path):
    out = str(tmp_path / "out.s")
    cmd = [build.hipcc_path()] + build.compile_flags() + ["-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return open(out).read()


def _kernels(text, name):
    """The bodies of the kernels whose mangled names contain `name`."""
    return [m.group(0) for m in re.finditer(r"^_ZN\w*" + name + r"\w*:.*?^\s*s_endpgm", text, flags=re.S | re.M)]


def test_ratio_kernels_load_four_tokens_at_a_time(tmp_path):
    try:
        build.hipcc_path()
    except RuntimeError:
        pytest.skip("no hipcc")
    text = _assembly("is_ratio.hip", tmp_path)
    for name in ("is_ratio_kernel", "grpo_surrogate_kernel"):
        bodies = _kernels(text, name)
        assert len(bodies) == 2, name                        # with and without a mask
        for body in bodies:
            # the current log-probs, and the old ones from either side of the stage boundary
            assert len(re.findall(r"global_load_dwordx4", body)) >= 3, name
