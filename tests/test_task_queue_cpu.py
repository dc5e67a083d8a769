"""The task queue of the one-launch selection (csrc/compams_tasks.h) on the host, threads for workgroups: every task once and in its
turn, also by a single workgroup, and every workgroup ends where the control blocks are written meanwhile."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2205_05632_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("queue") / "model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, os.path.join(HERE, "task_queue_model.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("disturb", [0, 1])
@pytest.mark.parametrize("workgroups,problems", [(1, 1), (1, 40), (3, 2), (8, 40), (24, 7)])
def test_every_wait_ends(model, workgroups, problems, disturb):
    for seed in range(5):
        r = subprocess.run([model, str(seed), str(workgroups), str(problems), str(disturb)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (seed, r.stdout, r.stderr)
