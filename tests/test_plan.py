"""The plans of a pass on the CPU: the arithmetic that the device runs (fpd_plan.hpp), compiled for
the host and checked against the sets of nodes it stands for.  Whatever the positions, the patch
kernel pulls only nodes that the step before updated, and the bead kernel pulls only nodes of the
step's set or nothing."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "plan")


def hipcc():
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    csrc = os.path.join(ROOT, "paper_2212_14153_amd", "csrc")
    subprocess.check_call([hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                           f"-I{csrc}", f"-I{os.path.join(ROOT, 'include')}",
                           os.path.join(HERE, "plan_check.cpp"), "-o", exe])
    return exe


def test_every_index_of_a_pass_lies_in_its_patch(program):
    out = subprocess.run([program, "3000"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:]
    words = out.stdout.split()
    seen = dict(zip(words[::2], map(int, words[1::2])))
    # every branch of the plan was met, beads inside and far outside it too
    assert all(n >= 20 for n in seen.values()), seen
