"""How the embedding and the GRU launches divide their work over workgroups (csrc/embed_rules.h, csrc/gru_rules.h), evaluated on
the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2308_14129_amd", "csrc")

WRAPPERS = """
#include "embed_rules.h"
#include "gru_rules.h"
extern "C" {
int gru_slices(int n_ct, int n_gru, int tiles) { return tig::column_slices(n_ct, n_gru, tiles).slices; }
int gru_holds(int n_ct, int n_gru, int guessed, int tiles) { return tig::slices_hold(tig::column_slices(n_ct, n_gru, guessed), n_gru, tiles); }
int height(int fp32, int neg, int most_mt, int rows, int units) { return tig::embed_height(fp32, neg, most_mt, rows, units); }
int tiles(int n_rows, int height, int units, int loop) { return tig::tiles_in_use(n_rows, height, units, loop); }
int step_wgs(int most, int height, int units) { return tig::step_workgroups(most, height, units); }
int any_wgs(int most, int top, int units) { return tig::any_workgroups(most, top, units); }
int overwrite_wgs(int wins, int waves) { return tig::overwrite_workgroups(wins, waves); }
int beside(int n_prepare, int wins, int waves) { return tig::overwrite_beside(n_prepare, wins, waves); }
int layer_wgs(int most, int top, int units) { return tig::layer_workgroups(most, top, units); }
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


def possible(most):
    return sorted(set(range(1, most, max(1, most // 97))) | {most - 1, most} - {0})


@pytest.mark.parametrize("neg", [0, 1])
@pytest.mark.parametrize("most_mt", [1, 2, 3])
def test_layer_rounds_are_what_the_compute_units_need(rules, most_mt, neg):
    # no workgroup takes a second tile while there are compute units without one, whatever the tile's height
    for units in UNITS:
        for most in ROWS:
            loop = rules.layer_wgs(most, rules.height(1, neg, most_mt, most, units), units)
            assert 1 <= loop <= units
            for n in possible(most):
                h = rules.height(1, neg, most_mt, n, units)
                used = rules.tiles(n, h, units, loop)
                assert used * h >= n
                assert -(-used // loop) <= max(1, -(-(-(-n // h)) // units)), (units, most, h, n)


@pytest.mark.parametrize("neg", [0, 1])
@pytest.mark.parametrize("most_mt", [1, 2, 3])
def test_every_row_of_a_step_has_a_workgroup_at_the_height_the_kernel_takes(rules, most_mt, neg):
    for units in UNITS:
        for most in ROWS:
            top = rules.height(1, neg, most_mt, most, units)
            wgs = rules.any_wgs(most, top, units)
            for n in possible(most):
                h = rules.height(1, neg, most_mt, n, units)
                used = rules.tiles(n, h, units, 0)
                assert h <= top and used <= wgs and used * h >= n, (units, most, h, n)


def test_every_row_of_a_step_has_a_workgroup_at_the_height_the_host_takes(rules):
    for units in UNITS:
        for most in ROWS:
            for rows in estimates(most):
                h = rules.height(0, 1, 3, rows, units)
                wgs = rules.step_wgs(most, h, units)
                for n in {1, rows // 2, rows, most}:
                    used = rules.tiles(n, h, units, 0)
                    assert used <= wgs and used * h >= n


def test_only_negatives_lie_in_the_last_eight_of_24_rows(rules):
    # (row r of tile p is row p + tiles * r of the set, negatives last; the places of the others are a matter of timing)
    for units in UNITS:
        for count in [1, 2, 7, 300, 597, 1021, 1100, 1250, 1790, 2000, 4099]:
            for n_u in possible(2 * count):
                n = n_u + count
                assert rules.height(1, 0, 3, n, units) != 24
                if rules.height(1, 1, 3, n, units) == 24:
                    for loop in (0, 1, units // 2, units):
                        assert 16 * rules.tiles(n, 24, units, loop) >= n_u, (units, count, n_u)


def test_the_overwrite_has_the_wavefronts_it_needs(rules):
    # `left` events remain behind a batch of `count`: at most 31 workgroups prepare them, one for every sixteen entries
    for waves in (8, 16):
        for count in [1, 16, 200, 1000, 4000, 4096, 12000]:
            for left in sorted({0, 1, 8, 200, count // 2, count}):
                prepare = min(31, -(-2 * left // 16)) if left <= 4096 else 0
                for wins in sorted({1, count // 3, count, 2 * count} - {0}):
                    own = rules.overwrite_wgs(wins, waves)
                    n = prepare if rules.beside(prepare, wins, waves) else own
                    assert n >= own and 1 <= own <= 16
                    assert wins / (n * waves) <= max(4.0, wins / (16 * waves))
                    if left == count and count <= 4096:
                        assert n == prepare  # (in the middle of a stream)


def test_foreseen_column_slices_are_those_of_the_winners_found(rules):
    # the kernel keeps the launch's slices exactly if it would have come to the same, whatever the winners they were for
    for n_ct in [1, 2, 3, 7, 11, 16, 32]:
        for most in [1, 2, 13, 100, 500, 1000]:  # tiles of winners that the batch could have
            n_gru = min(256, most * n_ct)
            for tiles in possible(most):
                got = rules.gru_slices(n_ct, n_gru, tiles)
                assert 1 <= got <= n_ct and (got == 1 or tiles * got <= n_gru)
                for guessed in possible(most):
                    same = rules.gru_slices(n_ct, n_gru, guessed) == got
                    assert rules.gru_holds(n_ct, n_gru, guessed, tiles) == same, (n_ct, n_gru, tiles, guessed)
