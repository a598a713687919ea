"""The bounded search of a table entry (csrc/mrg_hyper.h) against its definition, on
the host: random margins up to the largest total, uniforms next to 0 and 1, at simple
fractions, and on both sides of steps of the distribution function.  The search may
leave an entry undecided, never decide it otherwise.
"""
import os
import re
import subprocess

import pytest

from conftest import ROOT


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hyper") / "hyper_search_xcheck")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_2201_06604_amd", "csrc"),
                    os.path.join(ROOT, "tests", "xcheck", "hyper_search_xcheck.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("cases,total,steps,most_undecided", [
    (200_000, 60, 2000, 0.2), (60_000, 2000, 500, 0.2), (6000, 20_000, 60, 0.2), (60, 1 << 20, 2, 0.5)])
def test_search_is_the_definition_or_undecided(binary, cases, total, steps, most_undecided):
    r = subprocess.run([binary, str(cases), str(total), "7", str(steps)], capture_output=True, text=True, timeout=300)
    seen, undecided, wrong = map(int, re.search(r"(\d+) cases, (\d+) undecided, (\d+) wrong", r.stdout).groups())
    assert r.returncode == 0 and wrong == 0, r.stdout
    assert undecided < most_undecided * seen, r.stdout  # it does decide
