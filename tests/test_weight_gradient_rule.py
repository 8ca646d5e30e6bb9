"""CPU check of the rule that sends a weight gradient to the dense product or to the sums of the lanes that hold the nonzeros
(csrc/sprnn_wgrad_rule.h), against the times of both on MI355X."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# rows, columns, batch: {timesteps: (lane sums, product) in us}, measured with either alone
MEASURED = {
    (2304, 2304, 4): {1: (9.3, 10.5), 16: (28.1, 14.3), 64: (82.4, 26.4), 256: (285.2, 73.6)},
    (1152, 1152, 4): {16: (19.2, 8.9), 256: (237.7, 38.6)},
    (2560, 2560, 8): {16: (46.5, 22.7), 256: (696.3, 185.7)},
    (4096, 4096, 4): {1: (9.7, 23.9), 4: (14.8, 23.8), 64: (125.8, 68.0), 256: (443.3, 213.8)},
    (5000, 5000, 1): {16: (20.4, 40.9), 256: (216.4, 109.8)},
    (5120, 5120, 4): {16: (36.7, 51.9), 64: (140.2, 108.3), 256: (521.0, 332.3)},
    (5760, 5760, 2): {64: (131.5, 85.9), 256: (459.9, 226.0)},
    (8192, 8192, 4): {16: (57.6, 113.6), 64: (205.4, 240.6)},
    (8192, 8192, 2): {16: (42.4, 85.5), 256: (611.8, 400.0)},
    (8192, 8192, 1): {16: (21.2, 85.3), 64: (65.0, 110.4)},
    (11520, 11520, 1): {16: (22.6, 162.5), 64: (77.5, 208.2), 256: (277.9, 451.5)},
    (20000, 20000, 1): {16: (40.1, 467.6), 64: (130.8, 597.4), 256: (475.3, 1294.6)},
    (20000, 20000, 2): {16: (78.1, 478.7), 256: (1166.6, 2295.9)},
    (40000, 40000, 1): {16: (63.2, 1788.0), 64: (216.5, 2310.6), 256: (828.5, 5176.0)},
    (4 * 1024, 1024, 8): {16: (29.5, 13.7), 256: (322.5, 109.5)},
    (4 * 2048, 2048, 8): {64: (141.0, 118.5), 256: (521.8, 398.2)},
    (4 * 4096, 4096, 2): {16: (44.0, 87.6), 64: (114.4, 156.5)},
    (4 * 6000, 6000, 1): {16: (22.9, 182.9), 64: (75.4, 233.7), 256: (268.0, 498.5)},
    (4 * 10000, 10000, 1): {16: (22.5, 474.6), 64: (73.7, 600.7), 256: (260.4, 1331.8)},
    (3 * 2048, 2048, 4): {64: (76.5, 51.5), 256: (271.2, 166.9)},
    (3 * 4096, 4096, 2): {16: (42.5, 70.8), 256: (386.9, 331.6)},
    (3 * 8192, 8192, 1): {16: (27.9, 243.5), 64: (72.4, 306.8), 256: (234.1, 667.2)},
}


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++ here")
    out = str(tmp_path_factory.mktemp("rule") / "rule")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I" + os.path.join(ROOT, "paper_1804_10223_amd", "csrc"),
                    os.path.join(ROOT, "tests", "weight_gradient_rule.cpp"), "-o", out], check=True)

    def ask(calls):
        text = "".join("%d %d 256 %d %d\n" % c for c in calls)
        return subprocess.run([out], input=text, capture_output=True, text=True, check=True).stdout.split()
    return ask


def test_the_faster_way_is_taken(route):
    calls = [(shape + (T,), times) for shape, at in MEASURED.items() for T, times in at.items()]
    for (call, (lanes, product)), got in zip(calls, route([c for c, _ in calls])):
        assert got == ("lanes" if lanes < product else "product"), (call, lanes, product)


def test_more_vectors_than_the_product_counts(route):
    # (two billion vectors of a layer of one unit, which the product is otherwise the way for)
    assert route([(1, 1, 8, 2 ** 28 - 64), (1, 1, 8, 2 ** 28), (1, 1, 1, 2 ** 31 - 1)]) == ["product", "lanes", "lanes"]
