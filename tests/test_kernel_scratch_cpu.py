"""The sums of the four-wave Chebyshev P2M stay in registers at every order and
number of densities: an index that is known only at run time puts them into
scratch memory (it took 36 of the 84 variants there; order 8, three densities,
512 leaves of 80 points: 32.5 instead of 18.7 us). The compiler's own report of
each kernel's scratch size is read; no GPU is needed."""

import os
import re
import subprocess

import pytest


@pytest.mark.slow
def test_four_wave_p2m_uses_no_scratch(tmp_path):
    from paper_1605_01715_amd import build as B

    out = subprocess.run([B.hipcc(), *B.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
                          "-c", os.path.join(B.CSRC, "chebyshev.hip"), "-o", str(tmp_path / "chebyshev.o")],
                         capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-2000:]
    name, scratch = None, {}
    for line in out.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m[1]
        elif (m := re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)) and "k_points_to_nodes4" in name:
            scratch[name] = int(m[1])
    assert len(scratch) == 84  # 7 orders, 1 to 4 densities, single, double and both layers
    assert not {k: v for k, v in scratch.items() if v}
