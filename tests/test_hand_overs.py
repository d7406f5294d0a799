"""The words by which the workgroups of a launch hand each other results (csrc/hands.hpp), in all orders of their operations: hand_overs.cpp runs the
header on the host.  Every launch's work is done by one workgroup alone, with the results of that launch, and leaves nothing that the next one with
the same tag, a replayed graph's, would take for its own."""
import os
import subprocess

import pytest


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    here = os.path.dirname(os.path.abspath(__file__))
    out = str(tmp_path_factory.mktemp("hand_overs") / "hand_overs")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-o", out, os.path.join(here, "hand_overs.cpp")])
    return out


# rows of one to four chunks; the same past the L2s throughout; levels of one or two such rows.  (With two workgroups that may both take a row, "levels" fails at its
# second seed, and with a level that two may choose at its fourth.)  And launches whose words another one overwrites meanwhile, which only
# have to end ("overlap").
@pytest.mark.parametrize("scenario,seeds", [("rows", 1000), ("apart", 1000), ("levels", 400), ("overlap", 600)])
def test_any_order_of_the_hand_overs(program, scenario, seeds):
    done = subprocess.run([program, scenario, str(seeds)], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stdout
