"""The per-block sums that the blocks of a launch hand to its last block are
reached through put() and get() alone, whose accesses go past the caches that
blocks do not share: a plain load or store of them does not compile."""
import os
import subprocess

import pytest

from paper_2108_07001_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")


@pytest.mark.parametrize("line,ok", [
    ("a.partials.put(1, 2.0);", True),
    ("*out = a.t2_partials.get(3, 0, 4);", True),
    ("a.partials[0] = 2.0;", False),
    ("*a.t2_partials = 2.0;", False),
    ("double* p = a.partials; p[0] = 2.0;", False),
    ("a.partials.p_[0] = 2.0;", False),
])
def test_block_sums_have_no_plain_access(tmp_path, line, ok):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "probe.hip"
    src.write_text('#include "device_common.h"\n'
                   "__global__ void probe(const air::DemapArgs a, double* out) { " + line + " }\n")
    r = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "--offload-device-only",
                        "-I", CSRC, str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr
