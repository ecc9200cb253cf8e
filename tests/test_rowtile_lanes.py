"""The rules by size of the row tiles, over measured tiles and pieces (MI355X).
Lanes of the stored product's row passes: never more than 3% slower than the
passes of 128 rows, nor 20% slower than the fastest shape.  Threads of a matrix
pool's piece: the faster of a wave and a workgroup.  CPU only."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# entry bytes, tiles, rows, us by lanes 8 / 16 / 32 / 64
MEASURED = [
    (8, 64, 64, 17.0, 22.1, 33.6, 43.7), (8, 256, 64, 168.3, 181.9, 189.3, 220.4),
    (8, 256, 64, 203.7, 191.1, 204.5, 233.7), (8, 128, 128, 126, 120, 124, 185),
    (8, 512, 256, 1861, 1601, 1664, 1973), (8, 2048, 256, 7854, 6774, 6223, 6833),
    (8, 512, 95, 1893, 1581, 1667, 1433), (8, 2048, 98, 2158, 1781, 1654, 1441),
    (8, 2048, 147, 4278, 3289, 2979, 3552), (8, 64, 157, 97, 84, 103, 159),
    (8, 256, 49, 208.3, 172.2, 121.4, 153.6), (8, 128, 27, 24.1, 22.4, 28.5, 47.0),
    (4, 256, 256, 451, 432, 552, 591), (4, 4096, 256, 9058, 7792, 7454, 7942),
    (4, 128, 49, 37.5, 36.3, 46.7, 83.9), (4, 256, 98, 137.6, 134.1, 102.4, 135.4),
    (4, 512, 128, 247.9, 254.4, 256.7, 296.6), (4, 1024, 147, 1138, 979, 1054, 867),
    (2, 1024, 64, 82.5, 101.8, 166.7, 321.7), (2, 2048, 256, 1637, 1723, 1946, 2265),
    (2, 128, 98, 36.9, 43.0, 73.4, 116.4), (2, 256, 147, 140.7, 138.2, 175.2, 273.4),
    (2, 1024, 147, 608.6, 620.1, 509.5, 737.1), (2, 256, 400, 723.0, 707.3, 698.2, 891.0),
    (2, 128, 400, 342.1, 376.2, 388.0, 574.6), (2, 64, 512, 159.6, 175.6, 260.3, 445.2),
    (2, 64, 512, 333.5, 289.2, 413.8, 706.7), (2, 128, 64, 19.9, 28.8, 49.9, 124.3),
]


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("lanes")
    (d / "t.cpp").write_text("""
#include <cstdio>
#include <cstdlib>
#include "rowtile_lanes.h"
int main(int n, char** a) {
    if (n == 4 && atoi(a[1]) < 2) {
        printf("%d\\n", (int)hmx::piece_by_wave(atoi(a[1]), atol(a[2]), atol(a[3])));
        return 0;
    }
    const int es = atoi(a[1]), R = 16 / es, need = (atoi(a[3]) + R - 1) / R;
    printf("%d %d\\n", hmx::rowtile_lanes(atol(a[2]), need, es), hmx::rowtile_lanes_tall(need, R));
}
""")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I",
                           os.path.join(ROOT, "paper_1708_09707_amd", "csrc"), str(d / "t.cpp"),
                           "-o", str(d / "t")])
    return lambda *a: [int(v) for v in subprocess.check_output([str(d / "t")] + [str(v) for v in a]).split()]


@pytest.mark.parametrize("es,tiles,rows,t8,t16,t32,t64", MEASURED)
def test_pick_over_measured_tiles(pick, es, tiles, rows, t8, t16, t32, t64):
    t = {8: t8, 16: t16, 32: t32, 64: t64}
    lanes, tall = pick(es, tiles, rows)
    assert t[lanes] <= 1.03 * t[tall]
    assert t[lanes] <= 1.2 * min(t.values())


@pytest.mark.parametrize("es", [8, 4, 2])
def test_pick_is_a_shape(pick, es):
    for tiles in (1, 31, 256, 5000, 1 << 20):
        for rows in (1, 2, 63, 64, 65, 1000, 100000):
            assert set(pick(es, tiles, rows)) <= {8, 16, 32, 64}


# near field, units a piece (of factors: a bound), pieces, us as a workgroup and as a wave
PIECES = [(1, 343, 1000000, 3115, 1240), (1, 637, 500000, 1180, 607), (1, 1225, 100000, 1448, 976),
          (1, 2450, 50000, 628, 463), (1, 3510, 60000, 581, 659), (1, 7050, 20000, 490, 531),
          (1, 19200, 30000, 2831, 3736), (1, 2048, 1500, 20, 28), (0, 511, 4000000, 2397, 1620),
          (0, 511, 900000, 1405, 1107), (0, 1024, 100000, 795, 943)]


@pytest.mark.parametrize("near,units,pieces,group,wave", PIECES)
def test_piece_threads(pick, near, units, pieces, group, wave):
    (by_wave,) = pick(near, units * pieces, pieces)
    assert by_wave == (wave < group)
