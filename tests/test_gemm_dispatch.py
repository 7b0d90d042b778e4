"""Which kernel the rule sends the products of the GPU tests to: every shape of sub-tile, piece and pair is among them."""
import ctypes
import os
import subprocess

import pytest

import paper_2508_20258_amd as swz
import test_gpu_parity as gpu
from paper_2508_20258_amd.binding import SwzParams

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_20258_amd", "csrc")
SUB_TILES = [(32, 32), (32, 64), (64, 64), (128, 64), (64, 128), (128, 128), (128, 256), (64, 32), (96, 128), (192, 128)]


@pytest.fixture(scope="module")
def dispatch(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemm")
    (d / "g.cpp").write_text('#include "gemm_dispatch.h"\nextern "C" {\n'
                             "void shape(int s, int* out) { out[0] = swz::kSubTiles[s].bm; out[1] = swz::kSubTiles[s].bn; }\nint count() { return swz::kSubTileCount; }\n"
                             "void launch(long long m, long long n, long long k, int mode, const swz_params* r, int gm, int gn, int* out) {\n"
                             "  const swz::GemmLaunch l = swz::gemm_launch(m, n, k, *r, gm, gn, r->group_m < gm ? r->group_m : gm, mode, true, 256);\n"
                             "  out[0] = l.sub; out[1] = l.pieces; out[2] = l.pair; }\n}\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "g.cpp"), "-o", str(d / "g.so")], check=True)
    lib = ctypes.CDLL(str(d / "g.so"))
    assert lib.count() == len(SUB_TILES)
    for i, s in enumerate(SUB_TILES):
        out = (ctypes.c_int * 2)()
        lib.shape(i, out)
        assert tuple(out) == s

    def launch(M, N, K, mode=2):
        p = swz.gemm_plan(M, N, K, num_xcd=8)
        r = SwzParams(p["bm"], p["bn"], p["bk"], p["group_m"], p["num_xcd"], 0, 0)
        out = (ctypes.c_int * 3)()
        lib.launch(*[ctypes.c_longlong(v) for v in (M, N, K)], mode, ctypes.byref(r), p["grid_m"], p["grid_n"], out)
        sub, pieces, pair = out
        return "pair" if pair else "whole" if sub < 0 else (("pieces",) if pieces else ()) + SUB_TILES[sub]
    return launch


def test_the_sub_tile_test_reaches_every_shape(dispatch):
    reached = {}
    for M, N in gpu.SUBTILE_SHAPES:
        for K in gpu.subtile_ks(M, N):
            reached.setdefault(dispatch(M, N, K), set()).add(K)
    for shape in SUB_TILES:
        if shape != (64, 32):                                   # with feeders only
            assert len(reached[shape]) >= 4 and max(reached[shape]) > 512, (shape, reached.get(shape))
    # less than two stages, where the rule takes the shape for them
    assert all(min(reached[s]) <= 72 for s in SUB_TILES if s != (64, 32))


def test_the_piece_test_reaches_quarters_and_halves_from_their_shortest_k_on(dispatch):
    reached = {}
    for M, N in gpu.PIECE_SHAPES:
        for K in gpu.piece_ks(M, N):
            reached.setdefault(dispatch(M, N, K), set()).add(K)
        assert dispatch(M, N, 8) == dispatch(M, N, 200) == "pair" and dispatch(M, N, 456) != "pair"
    assert reached[("pieces", 128, 128)] >= {360, 456, 576, 1032} and reached[("pieces", 128, 256)] >= {360, 456, 712}
