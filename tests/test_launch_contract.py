"""What the host code launches is what the kernels take (CPU only): tables by
value of at most 32 curves and as many tiles as one launch may have workgroups,
tile lists for everything else, and an instance that carries every tile's path
(tests/native/launch_checks.cpp, under the address and undefined-behaviour
sanitizers)."""
from __future__ import annotations

import os

from tests.test_sanitizers import ASAN, _build_and_run, _host_cmd


def test_launches_follow_the_kernels_contract(tmp_path):
    cmd = [os.path.join(os.path.dirname(c), "launch_checks.cpp") if c.endswith(".cpp") else c
           for c in _host_cmd()]
    assert "launch checks ok" in _build_and_run(tmp_path, "launch_checks", cmd, ASAN, [])
