"""Launch shapes of the tiled kernels (CPU: the host functions of kernels.hpp
in a small program; nothing is launched).

A launch's x extent holds fewer than 2^32 threads, so many tiles go along x
and y.  Every tile needs a workgroup, and workgroups without a tile cost:
they take the LDS and the places of those with work.
"""

from __future__ import annotations

import os
import subprocess

import pytest

from paper_2510_05361_amd import build

SOURCE = r"""
#include <cstdio>
#include "kernels.hpp"
int main(int argc, char** argv) {
  long long tiles;
  int group;
  if (argc > 1) {  // "resident": replicas, bytes loaded per element; "group": row length, bytes of an element
    const bool many = argc > 2 && argv[2][0] == '1', clip = argc > 3 && argv[3][0] == '1';
    const bool outer = argc > 4 && argv[4][0] == '1';
    while (scanf("%lld %d", &tiles, &group) == 2)
      printf("%d\n", argv[1][0] == 'r' ? mtdao::wave_resident((int)tiles, group, many, clip, outer)
                                       : mtdao::row_group(tiles, group));
    return 0;
  }
  while (scanf("%lld %d", &tiles, &group) == 2) {
    const dim3 g = group == 0 ? mtdao::tile_grid(tiles, 3) : mtdao::group_grid(tiles, group, 3);
    printf("%u %u %u\n", g.x, g.y, g.z);
  }
}
"""
ONE_ROW = 1 << 21  # tiles of the largest one-dimensional launch
# around one and several rows, 1.31B x 4 (pieces), 354M x 16 (step tiles), 2^40 elements
TILES = [1, 7, 8, 16, 58_296, 1_381_252, ONE_ROW - 1, ONE_ROW, ONE_ROW + 1, ONE_ROW + 8, 2 * ONE_ROW,
         2 * ONE_ROW + 1, 3 * ONE_ROW + 17, 5_121_800, 11_050_016, 1 << 31, (1 << 32) + 1]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("shapes")
    src, exe = d / "shapes.hip", d / "shapes"
    src.write_text(SOURCE)
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    subprocess.run([build.HIPCC, *flags, "-O1", "-w", "-I", os.path.dirname(build.SRC), "-o", str(exe), str(src)],
                   check=True, stderr=subprocess.DEVNULL)

    def run(cases, *args):
        out = subprocess.run([str(exe), *args], input="".join(f"{a} {b}\n" for a, b in cases), capture_output=True,
                             text=True, check=True, timeout=60).stdout
        return dict(zip(cases, (tuple(int(v) for v in line.split()) for line in out.splitlines())))
    return run


@pytest.fixture(scope="module")
def grids(program):
    return program([(t, g) for t in TILES for g in (0, 1, 8)])


@pytest.mark.parametrize("group", [0, 1, 8])
@pytest.mark.parametrize("tiles", TILES)
def test_grid_covers_the_tiles_and_little_more(grids, tiles, group):
    x, y, z = grids[tiles, group]
    span = 1 if group < 2 else 8 * group  # pieces are taken in whole groups of the 8 XCDs
    whole = (tiles + span - 1) // span * span
    assert z == 3 and x * 1024 < 1 << 32 and 1 <= y <= 65535
    assert x * y >= whole
    # x a multiple of 16 keeps a tile's XCD and parity; at most that rounding is empty
    assert (y == 1 and x == whole) or (x % 16 == 0 and x * y - whole < 17 * y)


@pytest.mark.parametrize("many", ["0", "1"])
@pytest.mark.parametrize("clip", ["0", "1"])
@pytest.mark.parametrize("outer", ["0", "1"])
def test_more_due_states_and_clipping_never_lower_the_limit(program, many, clip, outer):
    """Exchanging more states, reading gradients that the clip norm has just
    read, or the OuterOpt asks for as many workgroups per CU or more."""
    forms = [(k, b) for k in range(2, 17) for b in range(8, 29, 2)]
    base, here = program(forms, "resident"), program(forms, "resident", many, clip, outer)
    # (16 bytes, every state due, no clipping: two workgroups from six replicas on)
    low = {f: (base[f], here[f]) for f in forms if here[f][0] < 2 or (here[f] < base[f] and f[0] < 6)}
    assert not low, low


def test_fused_step_keeps_loads_in_flight(program):
    """The limit of workgroups per CU leaves every form of the fused step at
    least 40 KiB of loads in flight (four elements per lane), also those with
    few streams; one that left them 24 KiB took their rate down by a third."""
    forms = [(k, b) for k in range(2, 9) for b in range(8, 29, 2)]
    resident = program(forms, "resident")
    low = {f: n for f, (n,) in resident.items() if n * f[0] * 64 * 4 * f[1] < 40 << 10 and n * f[0] < 32 - f[0]}
    assert not low, low


def test_rows_on_whole_lines_take_pieces_in_turn(program):
    """Only rows that start inside a 128-byte line take groups of pieces per
    XCD (on whole lines they cost the fused step 3 % and the K = 16 mean 4 %)."""
    cases = [(P, b) for P in (40_000_000 + r for r in (0, 1, 4, 8, 16, 32, 64, 96)) for b in (2, 4)]
    for (P, b), (group,) in program(cases, "group").items():
        assert group == (1 if P * b % 128 == 0 else 8), (P, b)
