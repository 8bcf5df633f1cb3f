"""How a launch of least-squares teams ends where workgroups run out of patience: the kernel's own rules (csrc/lsq_team_end.hpp) in
a model of a team on the CPU, under random schedules."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1910_12308_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lsq_team_end") / "lsq_team_end")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "lsq_team_end.cpp"), "-o", exe], check=True)

    def call(*args):
        return subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, check=True).stdout.split()
    return call


@pytest.mark.parametrize("reducers", [1, 2, 4, 16])
def test_every_schedule_ends_and_every_slice_is_written(model, reducers):
    assert model(4000 if reducers < 16 else 500, reducers) == ["endless", "0", "unwritten", "0", "lost", "0", "misnumbered", "0"]


# The bound of a wait for totals that a claim says are there: it ends although they are not
@pytest.mark.parametrize("reducers", [1, 4])
def test_a_wait_for_totals_that_do_not_come_ends(model, reducers):
    out = model(500, reducers, "wrong")
    assert out[:2] == ["endless", "0"] and int(out[5]) > 100
