"""The rules of a transpose's launch: order, loads on their way, blocks of part lines."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_20258_amd", "csrc")
RR, XCD, XCD_GROUPM, SKEWED = 0, 1, 2, 6


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("transpose")
    (d / "t.cpp").write_text('#include "transpose_dispatch.h"\nextern "C" {\n'
                             "int paced(int tile, long long m, long long n, int mode) { return swz::load_pace(tile, m, n, mode).paced; }\n"
                             "int lds(int tile, long long m, long long n, int mode) { return swz::load_pace(tile, m, n, mode).lds; }\n"
                             "int paced32(long long m, long long n) { return swz::paced_tiles32(m, n); }\n"
                             "int sweep(long long m, long long n, int eb) { return swz::sweep_tiles(m, n, eb); }\n"
                             "int lines(long long m, long long n, int eb) { return swz::line_blocks(m, n, eb); }\n}\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    for f in (lib.paced, lib.lds):
        f.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    lib.paced32.argtypes = [ctypes.c_longlong] * 2
    for f in (lib.sweep, lib.lines):
        f.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return lib


@pytest.mark.parametrize("M,N,mode,paced", [(16384, 16384, XCD_GROUPM, 1), (16384, 16384, RR, 1), (16384, 16384, SKEWED, 0), (16384, 4096, XCD_GROUPM, 1),
                                            (16384, 2048, XCD_GROUPM, 0), (16384, 4608, XCD_GROUPM, 0), (8192, 16384, XCD_GROUPM, 0), (4096, 8192, XCD, 1),
                                            (4096, 8192, RR, 0), (8192, 4096, XCD, 0), (2048, 8192, XCD, 0), (10048, 7040, XCD_GROUPM, 0)])
def test_loads_of_tiles_of_128(rules, M, N, mode, paced):
    assert rules.paced(128, M, N, mode) == paced and rules.lds(128, M, N, mode) == 0


@pytest.mark.parametrize("M,N,mode,paced,lds", [
    (1024, 1024, SKEWED, 0, 0), (2944, 2848, SKEWED, 0, 0), (2944, 2856, SKEWED, 1, 0), (5056, 5000, SKEWED, 1, 0), (5056, 5000, XCD, 1, 0),
    (4096, 4096, SKEWED, 0, 0), (2048, 4096, SKEWED, 0, 0), (4160, 4096, XCD_GROUPM, 0, 0), (4096, 4160, SKEWED, 0, 0), (4352, 4096, SKEWED, 1, 0),
    (8192, 2176, SKEWED, 0, 24576), (8192, 8192, SKEWED, 0, 24576), (8192, 8192, XCD_GROUPM, 1, 0), (16384, 16384, XCD_GROUPM, 0, 24576), (4096, 4096, XCD, 0, 24576),
    (4160, 4096, XCD, 1, 0), (2176, 2408, RR, 0, 0), (2176, 2416, RR, 1, 0), (4096, 2560, RR, 1, 0), (4096, 4096, RR, 0, 24576),
    (24576, 672, SKEWED, 0, 24576), (24576, 640, SKEWED, 0, 0), (1408, 12288, SKEWED, 1, 0), (64, 184320, SKEWED, 1, 0), (1600, 8192, SKEWED, 0, 0)])
def test_loads_of_tiles_of_64(rules, M, N, mode, paced, lds):
    assert (rules.paced(64, M, N, mode), rules.lds(64, M, N, mode)) == (paced, lds)
    assert (rules.paced(32, M, N, mode), rules.lds(32, M, N, mode)) == (0, 0)


@pytest.mark.parametrize("M,N,elem_bytes,sweep", [(16384, 16384, 2, 1), (8192, 32768, 2, 0), (4096, 16384, 4, 0), (4096, 8192, 4, 1), (10048, 7040, 2, 1),
                                                  (2048, 8192, 2, 0), (2048, 8200, 2, 1), (1536, 4096, 2, 0), (1472, 4096, 2, 1), (4288, 4096, 2, 0), (4352, 4096, 2, 1), (1408, 12288, 2, 1), (64, 184320, 2, 1)])
def test_which_tiles_are_swept(rules, M, N, elem_bytes, sweep):
    assert rules.sweep(M, N, elem_bytes) == sweep


@pytest.mark.parametrize("M,N,paced", [(2048, 2300, 0), (2048, 2304, 1), (2048, 4028, 1), (2048, 4032, 0), (64, 64, 0), (8192, 8192, 0)])
def test_loads_of_four_byte_tiles(rules, M, N, paced):
    assert rules.paced32(M, N) == paced


SHORT, TALL, TALL_PACED = 0, 1, 2


@pytest.mark.parametrize("M,N,elem_bytes,blocks", [
    (64, 87376, 2, SHORT), (72, 87376, 2, TALL), (256, 40000, 2, TALL), (264, 40000, 2, SHORT), (272, 200000, 2, SHORT), (280, 40000, 2, TALL), (312, 200000, 2, SHORT),
    (320, 200000, 2, TALL), (1024, 4456, 2, TALL), (1032, 5576, 2, SHORT), (1032, 5592, 2, TALL_PACED), (1032, 10152, 2, TALL_PACED), (1032, 10168, 2, TALL),
    (3080, 4248, 2, TALL_PACED), (3080, 4256, 2, TALL), (8200, 600, 2, SHORT), (10000, 7000, 2, TALL), (8, 1 << 29, 2, SHORT),
    (48, 60000, 4, SHORT), (52, 60000, 4, TALL), (128, 60000, 4, TALL), (132, 60000, 4, SHORT), (184, 60000, 4, SHORT), (188, 60000, 4, TALL),
    (260, 16000, 4, TALL_PACED), (256, 16000, 4, TALL), (260, 15620, 4, TALL), (1000, 5240, 4, TALL_PACED), (1000, 5244, 4, TALL), (1004, 7308, 4, TALL_PACED),
    (1004, 7316, 4, TALL), (5800, 5804, 4, TALL)])
def test_blocks_into_part_lines(rules, M, N, elem_bytes, blocks):
    assert rules.lines(M, N, elem_bytes) == blocks
