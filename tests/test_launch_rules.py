"""Rules that split work over workgroups, compiled from the library's own header for the CPU and looked at for every batch size."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GEOMETRIES = {"84": 0, "paper": 1, "a3c": 2}
PROGRAM = r"""
#include <cstdio>
#include "paper_1803_02811_amd/csrc/arn_layout.h"
int main() {
    for (int g = 0; g < 3; ++g)
        for (int B = 1; B <= 16384; B += B < 8300 ? 1 : 61) {
            arn_config c{};
            c.num_actions = 18; c.num_atoms = 51; c.geometry = g;
            const arn::Dims d = arn::make_dims(&c);
            const arn::ConvBwdSplit s = arn::conv_bwd_split(d, B), free = arn::conv_bwd_split(d, B, 1 << 20, 1 << 20);
            printf("%d %d %d %d %d %d %d %d %d\n", g, B, s.spw1, s.spw2, s.spw3, free.spw1, free.spw2, free.spw3,
                   arn::fc_wgrad_units(d.feat, d.hid, B));
        }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """{(geometry, batch): (samples per workgroup of the three ranges of the convolutions' backward, the same without the bounds on
    the counts, hidden units per tile of the fc weight gradient)}"""
    at = tmp_path_factory.mktemp("rules")
    (at / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", ROOT, str(at / "rules.cpp"), "-o", str(at / "rules")], check=True, timeout=100)
    out = subprocess.run([str(at / "rules")], check=True, capture_output=True, text=True, timeout=100).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    return {r[:2]: (r[2:5], r[5:8], r[8]) for r in rows}


@pytest.mark.parametrize("geometry", GEOMETRIES)
def test_convolution_backward_is_one_round_and_its_bounds_cut_nothing(rules, geometry):
    """At most one workgroup per CU, and the bounds that the workspace sizes rely on are what the rule comes to by itself."""
    for (g, B), (spw, free, _) in rules.items():
        if g == GEOMETRIES[geometry]:
            ranges = spw if geometry != "a3c" else spw[:2]
            assert sum(-(-B // n) for n in ranges) <= 256, B
            assert spw == free, B


@pytest.mark.parametrize("B,spw", [(150, (1, 4, 4)), (560, (4, 10, 12)), (1000, (7, 16, 20)), (1500, (11, 24, 32))])
def test_convolution_backward_split_of_measured_batches(rules, B, spw):
    """84x84 batches at which other ratios of the ranges' times gave splits that were measured 2 to 15% slower."""
    assert rules[0, B][0] == spw


@pytest.mark.parametrize("geometry,first", [("84", 2433), ("paper", 1153), ("a3c", None)])
def test_fc_weight_tiles_change_where_the_gpu_tests_look(rules, geometry, first):
    """test_gradients_at_fc_weight_tile_edges takes these batches and the ones before them."""
    wide = [B for (g, B), (_, _, units) in rules.items() if g == GEOMETRIES[geometry] and units == 256]
    assert min(wide, default=None) == first
    assert first is None or set(wide) == {B for g, B in rules if g == GEOMETRIES[geometry] and B >= first}
