"""The order of the second launch of a layer normalisation of long rows: a rule on sizes, and the caller's mapping where it is named."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_20258_amd", "csrc")


@pytest.fixture(scope="module")
def dispatch_order(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "r.cpp").write_text('#include "row_dispatch.h"\nextern "C" int f(long long m, long long n, int chunks, int x, int named) {\n'
                             "  return swz::emit_in_dispatch_order(m, n, chunks, x, named != 0); }\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    lib = ctypes.CDLL(str(d / "r.so"))
    return lambda N, M=64, num_xcd=8, named=False: bool(lib.f(ctypes.c_longlong(M), ctypes.c_longlong(N), -(-N // 16384), num_xcd, int(named)))


@pytest.mark.parametrize("N", [98312, 131072, 600000, 1048576, 1 << 24])
def test_a_named_mapping_is_the_caller_s(dispatch_order, N):
    assert not dispatch_order(N, named=True)


def test_gamma_and_beta_that_an_l2_keeps(dispatch_order):
    assert dispatch_order(131072) and dispatch_order(1048576)
    assert not dispatch_order(98312) and not dispatch_order(600000)


def test_chunks_that_share_no_xcd_keep_the_caller_s_order(dispatch_order):
    assert not dispatch_order(800000) and not dispatch_order(2000000)          # 49 and 123 chunks on 8 XCDs
    assert dispatch_order(850000) and dispatch_order(1000000)                  # 52, 62
    assert not dispatch_order(1048576, num_xcd=1)


def test_chunks_that_cut_lines(dispatch_order):
    assert dispatch_order(114696, M=292) and not dispatch_order(114696, M=293)       # 2^25 elements lie between
    assert not dispatch_order(250000, M=256) and not dispatch_order(131064, M=1024)
    assert dispatch_order(131072, M=1024) and dispatch_order(1048568, M=1024)        # chunks on lines; gamma and beta beyond 3 MiB
