"""What bench.py says of a mapping of several parts (CPU): its bound is that of a part's share of the samples, its labels are those
of the kernel that runs, and counters of another kernel are not quoted."""
import importlib.util
import os
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROBES = {"lds_Bps": {4: 70e12, 8: 140e12, 16: 150e12}, "valu_lane_ops_per_s": 39e12, "handoff_same_ns": 320.0, "handoff_cross_ns": 400.0,
          "fill_s_per_byte": 1 / 114e9}


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


def test_the_bound_of_several_parts_is_that_of_a_parts_share(bench):
    w = SimpleNamespace(hidden=2304, batch=4, nnz=2304 * 691)
    one, two = (bench.roofline_for(w, {"parts": n, "grid": 256 // n, "one_xcd": 0}, PROBES) for n in (1, 2))
    assert one["h_bytes"] == 2304 * 16 and two["h_bytes"] == 2304 * 8 and two["t_fill_us"] == pytest.approx(one["t_fill_us"] / 2)
    assert one["lds_bytes_per_step"] == two["lds_bytes_per_step"] == w.nnz * 16     # every part gathers for every nonzero
    assert two["t_lds_us"] == pytest.approx(w.nnz * 16 / 140e12 * 1e6)              # ... 8 bytes at a time
    assert two["t_roof_us"] < one["t_roof_us"]
    assert bench.kernel_label(w, {"parts": 2, "template_words": 24}) == "persistent_kernel<B=2,NW=24>"


def test_counters_of_another_kernel_are_not_quoted(bench, tmp_path):
    path = tmp_path / "traffic.txt"
    path.write_text("workload = cfg3\nkernel = void sprnn::persistent_kernel<2, 24, 0, false, 2>(sprnn::KernelArgs)\n"
                    "fetch_bytes_per_launch = 1000\nwrite_bytes_per_launch = 500\n")
    assert bench.read_traffic_file(str(path), "cfg3", 2, 24)["fetch_bytes_per_launch"] == 1000.0
    assert bench.read_traffic_file(str(path), "cfg3", 4, 16) is None
    assert bench.read_traffic_file(str(path), "cfg2", 2, 24) is None
