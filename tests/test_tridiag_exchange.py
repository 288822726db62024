"""CPU model of the exchange between the workgroups of the in-register
tridiagonal reduction (csrc/tridiag.hip): the rules of csrc/tridiag_steps.hpp,
which the kernel is built from, under schedules that hold any workgroup's reads
in any step, and under random ones.  Nobody may wait for ever, whatever the
delays; with a workgroup that still reads in its last step somebody does."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_00079_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("exchange") / "model")
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", "-o", exe,
                    os.path.join(HERE, "tridiag_exchange_model.cpp")], check=True)

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        runs, stuck = map(int, r.stdout.split())
        return runs, stuck
    return run


# whole and ragged last workgroups (one row, two, seven), a single workgroup
@pytest.mark.parametrize("n", [3, 8, 9, 10, 15, 16, 17, 64, 71])
def test_nobody_waits_for_ever(model, n):
    runs, stuck = model(0, n, n, 40)
    assert runs > 40 and stuck == 0


def test_the_model_sees_a_late_leaver(model):
    runs, stuck = model(1, 64, 1, 0)
    # at least where one of the seven that leave is held in its last step
    assert stuck >= 7 * 3, (runs, stuck)
