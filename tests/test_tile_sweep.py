"""The order in which a transpose sweeps its tiles: every tile once, whatever the grid, the XCD count and the rows of an XCD."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_20258_amd", "csrc")


@pytest.fixture(scope="module")
def sweep(tmp_path_factory):
    d = tmp_path_factory.mktemp("sweep")
    (d / "s.cpp").write_text('#include "tile_sweep.h"\nextern "C" void sweep(int gm, int gn, int x, int rows, int* out) {\n'
                             "  for (int w = 0, pm, pn; w < gm * gn; ++w) { swz_sweep_tile(w, gm, gn, x, rows, &pm, &pn); out[2 * w] = pm; out[2 * w + 1] = pn; } }\n"
                             'extern "C" int rows(int gm, int x, int eb) { return swz_sweep_rows(gm, x, eb); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))

    def tiles(gm, gn, x, rows):
        out = np.full((gm * gn, 2), -1, dtype=np.int32)
        lib.sweep(gm, gn, x, rows, out.ctypes.data_as(ctypes.c_void_p))
        return out
    tiles.rows = lib.rows
    return tiles


# windows without a rest, with one row and with all but one row left, none at all; fewer rows than XCDs
@pytest.mark.parametrize("gm", [1, 2, 7, 8, 9, 24, 31, 32, 33, 46, 63, 64, 65, 127])
@pytest.mark.parametrize("gn", [1, 2, 13, 91])
def test_every_tile_once(sweep, gm, gn):
    for x in (1, 3, 8, 1000):
        for rows in sorted({1, 2, 4, sweep.rows(gm, x, 2), sweep.rows(gm, x, 4)}):
            t = sweep(gm, gn, x, rows)
            assert (t >= 0).all() and (t[:, 0] < gm).all() and (t[:, 1] < gn).all()
            assert len(np.unique(t[:, 0].astype(np.int64) * gn + t[:, 1])) == gm * gn, (x, rows)


def test_an_xcd_keeps_its_rows_of_a_window_and_sweeps_the_columns(sweep):
    gm, gn, x, rows = 70, 11, 8, 4                 # two windows of 32 rows, six rows left
    t = sweep(gm, gn, x, rows)
    for w in range(64 * gn):
        win, k = divmod(w, 32 * gn)
        assert t[w, 0] // 4 == win * 8 + w % 8 and t[w, 1] == k // 8 // 4
    assert (t[64 * gn:, 0] >= 64).all()
