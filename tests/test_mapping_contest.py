"""Which mapping sprnn_create keeps (csrc/sprnn_contest.h), on the CPU with made-up times and failures: a creation that can succeed
does, no call is lost to a faster mapping, and a handle of several parts has one with the same lanes behind it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ALL = (1, 1, 1, 1)


def made(parts, lanes, us, can=ALL, grid=0, compact=0, proposed=0):
    return (parts, lanes, grid, compact, us) + tuple(can) + (proposed,)


@pytest.fixture(scope="module")
def contest(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("contest") / "contest")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1804_10223_amd", "csrc"),
                    os.path.join(ROOT, "tests", "mapping_contest.cpp"), "-o", exe], check=True)

    def run(batch, mappings, most_lanes=64):
        text = "%d %d\n" % (batch, most_lanes) + "\n".join(" ".join(map(str, m)) for m in mappings)
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout
        line = lambda word: next((tuple(map(float, re.findall(r"[\d.]+", l))) for l in out.splitlines() if l.startswith(word)), None)
        assert line("left") == (0,), out
        return line("kept"), line("behind"), out.count("asked")
    return run


def test_the_packers_own_mapping_is_kept_when_nothing_else_can_be_had(contest):
    assert contest(8, [made(1, 32, 2.0, proposed=9)]) == ((1, 32, 0, 2.0), None, 1 + 2 + 3)


@pytest.mark.parametrize("own", [2.0, 0.9])
def test_a_division_has_the_fastest_handle_of_its_lanes_behind_it(contest, own):
    # other lanes than the packer's own win; the handle behind is the one that was measured: nothing is built once a division
    # was kept, so nothing can fail any more
    kept, behind, asked = contest(4, [made(1, 64, own), made(1, 32, 2.5), made(2, 32, 0.8), made(4, 32, 0.7)])
    assert kept == (4, 32, 0, 0.7) and behind == (1, 32, 0, 2.5) and asked == 1 + 2 + 2
    kept, behind, _ = contest(4, [made(1, 32, own), made(2, 32, 0.8)])
    assert kept == (2, 32, 0, 0.8) and behind == (1, 32, 0, own)


def test_a_division_into_lanes_without_a_handle_behind_is_not_kept(contest):
    assert contest(2, [made(1, 64, 2.0), made(2, 32, 0.5)])[:2] == ((1, 64, 0, 2.0), None)
    # ... nor where that handle copies only the columns its rows read
    assert contest(2, [made(1, 64, 2.0), made(1, 32, 2.1, compact=1), made(2, 32, 0.5)])[:2] == ((1, 64, 0, 2.0), None)


@pytest.mark.parametrize("lost", range(4))
def test_no_call_is_lost_to_a_faster_mapping(contest, lost):
    less = tuple(0 if i == lost else 1 for i in range(4))
    # one part, other lanes
    assert contest(1, [made(1, 32, 2.0), made(1, 16, 1.0, can=less)])[:2] == ((1, 32, 0, 2.0), None)
    # ... or fewer workgroups
    assert contest(1, [made(1, 32, 2.0, proposed=5), made(1, 32, 1.0, can=less, grid=5)])[:2] == ((1, 32, 0, 2.0), None)
    # a division whose lanes only a handle without that call has
    assert contest(2, [made(1, 32, 2.0), made(1, 16, 3.0, can=less), made(2, 16, 1.0)])[:2] == ((1, 32, 0, 2.0), None)
    # a division: the weight gradients are those of the handle behind it, the other calls its own
    kept, behind, _ = contest(2, [made(1, 32, 2.0), made(2, 32, 1.0, can=less)])
    assert (kept, behind) == (((2, 32, 0, 1.0), (1, 32, 0, 2.0)) if lost in (1, 2) else ((1, 32, 0, 2.0), None))
    # what the packer's own mapping cannot do, the others need not
    assert contest(1, [made(1, 32, 2.0, can=less), made(1, 16, 1.0, can=less)])[0] == (1, 16, 0, 1.0)


def test_the_fastest_is_kept(contest):
    assert contest(1, [made(1, 16, 2.0, proposed=7), made(1, 16, 1.5, grid=7), made(1, 32, 1.4), made(1, 8, 1.45)])[0] == (1, 32, 0, 1.4)
    assert contest(1, [made(1, 16, 2.0), made(1, 32, 1.99)])[0] == (1, 16, 0, 2.0)              # within two per cent: the packer's
    kept, behind, _ = contest(8, [made(1, 16, 2.0, proposed=7), made(1, 16, 1.5, grid=7), made(2, 16, 1.4), made(4, 16, 1.2, proposed=3),
                                  made(4, 16, 1.1, grid=3), made(8, 16, 1.3)])
    assert kept == (4, 16, 3, 1.1) and behind == (1, 16, 7, 1.5)
    assert contest(4, [made(1, 16, 2.0), made(2, 16, 0.0)])[0] == (1, 16, 0, 2.0)                # not measured
