"""What works where the extension module of the per-step calls cannot be had."""
import os
import subprocess
import sys

from paper_2605_10670_amd import build


def test_host_only_calls_do_without_the_module():
    """No module and no compiler: planners and sizes work, a per-step call says what is missing."""
    code = """
import sys
sys.modules["paper_2605_10670_amd._marshal"] = None
import numpy as np
from paper_2605_10670_amd import binding, build
build.MARSHAL = "/nonexistent/module.so"
assert binding.workspace_bytes(num_ranks=2, slots_per_rank=4, primary_slots=4, num_logical=8, max_tokens=8,
                               topk=2, hidden=64) > 0
assert binding.plan_repair(np.arange(8) % 8, np.ones(2), 2, 4, 4, 8)["status"] == binding.OK
try:
    binding._call(0, "h", 0)
except RuntimeError as e:
    assert "could not be built" in str(e)
else:
    raise AssertionError("called without a module")
"""
    env = dict(os.environ, CXX="/bin/false")
    subprocess.run([sys.executable, "-c", code], check=True, env=env, cwd=build.ROOT)
