"""The exchange of the tridiagonalisation's workgroups ends under any delay of a workgroup: a host
model (tridiag_exchange_model.cpp) of the two alternating sets of slots, run with the kernel's own
rule of who reads a column (csrc/tridiag_exchange.h).  The model finds the waits without end that
other rules allow: a workgroup without a row left keeps reading, or one reads the last column in
which it has a row."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2302_09708_amd", "csrc")

# (groups, n): more rows than groups, remainders, the kernel's own counts at n = 130 and 160
SIZES = [(2, 5), (3, 17), (5, 16), (8, 33), (9, 130), (10, 160)]


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("exchange") / "model")
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "tridiag_exchange_model.cpp"), "-o", exe],
                   check=True)

    def run(rule, groups, n):
        out = subprocess.run([exe, str(rule), str(groups), str(n)], check=True, capture_output=True, text=True).stdout
        _, _, _, runs, stuck = (int(v) for v in out.split())
        assert runs == 3 * groups * (n - 1) + 200
        return stuck

    return run


@pytest.mark.parametrize("groups,n", SIZES)
def test_every_wait_ends(model, groups, n):
    assert model(0, groups, n) == 0


@pytest.mark.parametrize("rule", [1, 2])
@pytest.mark.parametrize("groups,n", SIZES[1:])  # with two workgroups no slot of an idle one is written over
def test_the_model_finds_waits_without_end(model, rule, groups, n):
    assert model(rule, groups, n) > 0
