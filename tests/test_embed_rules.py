"""How an embedding launch divides its rows over workgroups (csrc/embed_rules.h), evaluated on the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2308_14129_amd", "csrc")

WRAPPERS = """
#include "embed_rules.h"
extern "C" {
int height(int fp32, int most_mt, int rows, int units) { return tig::embed_height(fp32, most_mt, rows, units); }
int tiles(int n_rows, int height, int units, int loop) { return tig::tiles_in_use(n_rows, height, units, loop); }
int step_wgs(int most, int height, int units) { return tig::step_workgroups(most, height, units); }
int layer_wgs(int most, int height, int units) { return tig::layer_workgroups(most, height, units); }
}
"""

ROWS = [1, 3, 4, 9, 33, 299, 300, 600, 895, 900, 1021, 1024, 1500, 1801, 2040, 4099, 6000, 12000, 66000]
UNITS = [16, 224, 255, 256]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "rules.so"), str(d / "rules.cpp")],
                   check=True)
    return ctypes.CDLL(str(d / "rules.so"))


def estimates(most):
    return sorted({most, max(1, most * 9 // 10), max(1, most // 2), max(1, most // 7)})


@pytest.mark.parametrize("most_mt", [1, 2, 3])
def test_layer_rounds_are_what_the_compute_units_need(rules, most_mt):
    # no workgroup takes a second tile while there are compute units without one, whatever the tile's height
    for units in UNITS:
        for most in ROWS:
            for rows in estimates(most):
                h = rules.height(1, most_mt, rows, units)
                loop = rules.layer_wgs(most, h, units)
                assert 1 <= loop <= units
                for n in {1, rows // 2, rows}:
                    used = rules.tiles(n, h, units, loop)
                    assert used * h >= n
                    assert -(-used // loop) <= max(1, -(-(-(-n // h)) // units)), (units, most, rows, h, n)


@pytest.mark.parametrize("fp32", [0, 1])
def test_every_row_of_a_step_has_a_workgroup(rules, fp32):
    for units in UNITS:
        for most in ROWS:
            for rows in estimates(most):
                h = rules.height(fp32, 3, rows, units)
                wgs = rules.step_wgs(most, h, units)
                for n in {1, rows // 2, rows, most}:
                    used = rules.tiles(n, h, units, 0)
                    assert used <= wgs and used * h >= n
