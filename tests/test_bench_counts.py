"""The benchmark's roofline counts the rule that the kernels evaluate (host)."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_counts_of_the_piece_form(bench):
    # a run's crossing: 24 for the form and 26 for its integral take the place of
    # the Gauss rule's 102 with scale, which leaves 4 + 6 beside them
    assert bench.RUN_FLOPS_PER_CROSSING == {"fp32": 112, "fp64": 8}
    # its transpose: 76 take the place of the three nodes' 114
    assert bench.ADJ_RUN_FLOPS_PER_CROSSING == {"fp32": 124, "fp64": 9}


def test_rooflines_use_them():
    with open(os.path.join(ROOT, "bench.py")) as f:
        text = f.read()
    used = [line for line in text.split("\n") if "flops_eq =" in line]
    assert len(used) == 2 and all("RUN_FLOPS_PER_CROSSING" in line for line in used)
