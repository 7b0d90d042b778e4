"""Host-side checks of libswz that need no GPU: exports, the closed-form PID map, error paths."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2508_20258_amd as swz
from oracle import pid_map as opm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_entry_point():
    header = open(os.path.join(ROOT, "include", "swz.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(swz_[a-z_]+)\s*\(", header))
    assert declared == {"swz_status_string", "swz_device_info", "swz_pid_map", "swz_pid_map_device", "swz_gemm",
                        "swz_gemm_ex", "swz_gemm_plan", "swz_copy_bytes", "swz_pid_map_persistent",
                        "swz_pid_map_persistent_device", "swz_transpose", "swz_softmax", "swz_layernorm", "swz_mfma_peak",
                        "swz_gemm_probe", "swz_gemm_launch_map"}
    raw = ctypes.CDLL(swz.binding.LIB_PATH)
    for name in declared:
        assert hasattr(raw, name), name
    assert set(swz.binding.EXPORTS) == declared


GRIDS = [(gm, gn) for gm in range(1, 13) for gn in range(1, 13)]


@pytest.mark.parametrize("mode", [0, 1, 2, 3, 4, 5, 6, 7])
def test_closed_form_equals_constructive_oracle_exhaustively(mode):
    for gm, gn in GRIDS:
        for X in range(1, 13):
            for g in range(1, 14):
                got = swz.pid_map(gm, gn, X, g, mode).tolist()
                assert got == opm.pid_map(gm, gn, X, g, mode), (gm, gn, X, g, mode)


@pytest.mark.parametrize("gm,gn,X,g", [(4, 4, 8, 4), (16, 16, 8, 4), (32, 32, 8, 4), (64, 8, 8, 4), (40, 28, 8, 4),
                                       (79, 55, 8, 4), (79, 28, 8, 4), (5, 5, 8, 4), (7, 3, 8, 4), (4, 5, 4, 4),
                                       (128, 96, 8, 16), (65, 67, 7, 5), (1, 300, 8, 4), (300, 1, 8, 4)])
def test_workload_grids_match_oracle_and_invariants(gm, gn, X, g):
    for mode in range(8):
        got = swz.pid_map(gm, gn, X, g, mode).tolist()
        assert got == opm.pid_map(gm, gn, X, g, mode)
        renumber, grouped, skewed = opm.mode_parts(mode)
        assert opm.is_permutation(got, gm * gn) and opm.fair_share(got, gm, gn, g, grouped, X, renumber, skewed)
        if renumber:
            assert opm.xcd_runs_contiguous(got, gm, gn, g, grouped, X, skewed)


def test_error_paths_leave_output_untouched():
    L = swz.lib
    out = np.full(16, -7, dtype=np.int32)
    for args in [(0, 4, 8, 4, 0), (4, 0, 8, 4, 0), (4, 4, 0, 4, 1), (4, 4, 8, 0, 2), (4, 4, 8, 4, 8), (4, 4, 8, 4, -1),
                 (-3, 4, 8, 4, 0)]:
        assert L.swz_pid_map(*args, out.ctypes.data) == -1
        assert (out == -7).all()
    assert L.swz_pid_map(4, 4, 8, 4, 0, None) == -1
    assert L.swz_pid_map(1 << 16, 1 << 15, 8, 4, 0, out.ctypes.data) == -3       # 2^31 tiles
    assert (out == -7).all()
    with pytest.raises(swz.SwzError) as e:
        swz.pid_map(4, 4, 8, 4, 9)
    assert e.value.status == -1
    assert swz.status_string(0) == "ok" and "unknown" in swz.status_string(-99)
    for s in (-1, -2, -3, -4):
        assert swz.status_string(s) and "unknown" not in swz.status_string(s)


def test_launches_of_2_to_the_32_threads_are_refused():
    # the device takes a grid in threads modulo 2^32: such a launch would run a remainder of it and report success
    L = swz.lib
    p = ctypes.byref(swz.SwzParams(0, 0, 0, 0, 8))
    a, b = 0x1000, 0x2000                  # never dereferenced
    for gm, gn in [(1 << 13, 1 << 13), (1 << 13, (1 << 13) + 1)]:
        assert L.swz_pid_map_device(gm, gn, 8, 4, 0, a, None, None) == -3
    assert L.swz_pid_map_persistent_device(4, 4, 8, 4, 0, (1 << 26) + 1, a, None, None) == -3
    assert L.swz_transpose(a, b, 8, (1 << 30) + 8, 2, 64, 2, p, None) == -3
    assert L.swz_transpose(a, b, 1 << 17, 1 << 17, 2, 32, 0, p, None) == -3
    assert L.swz_transpose(a, b, 4, (1 << 30) + 4, 4, 64, 2, p, None) == -3


# fewer than 2^24 tiles of 64 x 64 are never too many, whatever blocks they are done in: 8 rows of `out` off their lines, one row of tiles (and
# three, which are two blocks of four-byte elements)
@pytest.mark.parametrize("M,N,elem_bytes", [(8, 1 << 29, 2), (8, 1 << 29, 4), (60, 1 << 29, 4), (164, 1 << 28, 4), (8, (1 << 30) - 64, 2), (4, (1 << 30) - 64, 4)])
def test_transposes_of_fewer_than_2_to_the_24_tiles_are_not_refused(M, N, elem_bytes):
    import torch
    if torch.cuda.device_count() > 0:
        pytest.skip("the pointers are not real: for a machine where the launch itself fails")
    p = ctypes.byref(swz.SwzParams(0, 0, 0, 0, 8))
    assert -(-M // 64) * -(-N // 64) < 1 << 24
    assert swz.lib.swz_transpose(0x1000, 0x2000, M, N, elem_bytes, 64, 2, p, None) == -4          # no device


def test_long_rows_refuse_overlapping_buffers():
    # rows above 98304 elements keep statistics in the output while the input is read again: in place they would come out wrong
    L = swz.lib
    p = ctypes.byref(swz.SwzParams(0, 0, 0, 0, 8))
    x, M, N = 1 << 20, 3, 98312
    for out in (x, x + 16, x + 2 * (M * N - 8), x - 16):
        assert L.swz_softmax(x, out, M, N, 1, 1, p, None) == -1
        assert L.swz_layernorm(x, x, x, out, M, N, 1e-5, 1, 1, p, None) == -1


def test_group_m_larger_than_grid_is_one_band():
    assert swz.pid_map(5, 7, 8, 1 << 30, 3).tolist() == opm.pid_map(5, 7, 8, 5, 3)


def test_plan_resolves_tiles_without_a_device_when_num_xcd_is_given():
    p = swz.gemm_plan(512, 512, 512, num_xcd=8)
    assert (p["bm"], p["bn"], p["bk"], p["grid_m"], p["grid_n"], p["group_m"]) == (128, 128, 64, 4, 4, 4)
    p = swz.gemm_plan(10000, 7000, 4096, num_xcd=8)
    assert (p["bm"], p["grid_m"], p["grid_n"]) == (256, 40, 28)
    # grids far from the device's CU count are decided without asking a device: tiny -> 128-wide, huge -> 256-wide
    assert swz.gemm_plan(1024, 1024, 64, num_xcd=8)["bm"] == 128 and swz.gemm_plan(8192, 8192, 64, num_xcd=8)["bm"] == 256
    p = swz.gemm_plan(10000, 7000, 4096, num_xcd=8, bm=128, bn=256)
    assert (p["bm"], p["bn"], p["grid_m"], p["grid_n"]) == (128, 256, 79, 28)
    p = swz.gemm_plan(10000, 7000, 4096, num_xcd=8, bm=256, bn=128)
    assert (p["grid_m"], p["grid_n"]) == (40, 55)
    p = swz.gemm_plan(10000, 7000, 4096, num_xcd=8, bm=128, bn=128)
    assert (p["grid_m"], p["grid_n"]) == (79, 55)
    for bad in [dict(bm=64, bn=64), dict(bm=256, bn=64), dict(bm=512, bn=256), dict(bk=32)]:
        with pytest.raises(swz.SwzError) as e:
            swz.gemm_plan(1024, 1024, 1024, num_xcd=8, **bad)
        assert e.value.status == -2
    with pytest.raises(swz.SwzError) as e:
        swz.gemm_plan(0, 8, 8, num_xcd=8)
    assert e.value.status == -1
    with pytest.raises(swz.SwzError) as e:
        swz.gemm_plan(1 << 31, 8, 8, num_xcd=8)
    assert e.value.status == -3


def covers_once(blocks, M, N):
    count = np.zeros((M, N // 8), dtype=np.int32)
    for row, col, rows, cols in blocks[blocks[:, 2] > 0]:
        assert 0 <= row and row + rows <= M and 0 <= col and col + cols <= N and col % 8 == cols % 8 == 0
        count[row:row + rows, col // 8:(col + cols) // 8] += 1
    return bool((count == 1).all())


# sub-tiles of every shape, halves and quarters of the last round (with fewer left-over tiles than XCDs and more), whole tiles
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (100, 520, 64), (300, 1032, 64), (449, 1992, 512), (1217, 1544, 512), (300, 5000, 512), (1537, 1400, 512),
                                   (40, 33000, 200), (70, 66000, 512), (4352, 4096, 512), (1800, 9472, 64), (5120, 4608, 512), (4610, 5000, 64),
                                   (65793, 248, 64), (4096, 4096, 4096), (5120, 5120, 512),
                                   (1800, 9472, 704), (4610, 5000, 704), (65793, 248, 704), (4352, 4096, 704),
                                   (577, 3848, 512), (1537, 2680, 512), (193, 12304, 512)])
def test_launch_map_covers_c_once(M, N, K):
    for mode, params in [(0, dict(num_xcd=8)), (2, dict(num_xcd=8)), (1, dict(num_xcd=3)), (6, dict(num_xcd=8, group_m=3)), (5, dict(num_xcd=1000)),
                         (2, dict(num_xcd=1)), (2, dict(num_xcd=8, bm=128, bn=256))]:
        blocks = swz.gemm_launch_map(M, N, K, mode, **params)
        assert covers_once(blocks, M, N), (mode, params)


def test_launch_map_of_tiles_subtiles_and_pieces():
    # whole tiles: the plan's grid under swz_pid_map; sub-tiles: the same of a finer grid with a band as high; pieces: on the XCD of their tile
    def tiles(blocks, bm, bn, gn):
        return (blocks[:, 0] // bm * gn + blocks[:, 1] // bn).tolist()

    p = swz.gemm_plan(10000, 7000, 4096, num_xcd=8, bm=256, bn=256)
    got = swz.gemm_launch_map(10000, 7000, 4096, 2, num_xcd=8, bm=256, bn=256)
    assert tiles(got, 256, 256, p["grid_n"]) == opm.pid_map(p["grid_m"], p["grid_n"], 8, 4, 2)
    got = swz.gemm_launch_map(512, 512, 512, 2, num_xcd=8)
    assert len(got) == 256 and (got[:, 2:] == 32).all() and tiles(got, 32, 32, 16) == opm.pid_map(16, 16, 8, 16, 2)
    got = swz.gemm_launch_map(10000, 7000, 4096, 2, num_xcd=8)
    whole = opm.pid_map(40, 28, 8, 4, 2)
    assert tiles(got[:1024], 256, 256, 28) == whole[:1024]
    xcd_of_tile = {t: w % 8 for w, t in enumerate(whole)}
    for w, (row, col, rows, cols) in enumerate(got[1024:].tolist(), 1024):
        assert rows == 0 or (rows <= 128 and w % 8 == xcd_of_tile[row // 256 * 28 + col // 256])


def test_launch_map_error_paths():
    L, n = swz.lib, ctypes.c_int64(-7)
    p, out = ctypes.byref(swz.SwzParams(0, 0, 0, 0, 8)), np.full(8, -7, dtype=np.int32)
    ref = ctypes.byref(n)
    assert L.swz_gemm_launch_map(64, 64, 64, 0, p, None, 0, None) == -1
    assert L.swz_gemm_launch_map(64, 64, 64, 8, p, None, 0, ref) == -1
    assert L.swz_gemm_launch_map(0, 64, 64, 0, p, None, 0, ref) == -1
    assert L.swz_gemm_launch_map(64, 60, 64, 0, p, None, 0, ref) == -2
    assert L.swz_gemm_launch_map(64, 64, 64, 0, p, out.ctypes.data, 8, ref) == -1         # four sub-tiles
    assert L.swz_gemm_launch_map(1 << 31, 64, 64, 0, p, None, 0, ref) == -3
    persistent = swz.SwzParams(0, 0, 0, 0, 8, 1, 256)
    assert L.swz_gemm_launch_map(64, 64, 64, 0, ctypes.byref(persistent), None, 0, ref) == -2
    assert n.value == -7 and (out == -7).all()


def test_gemm_rejects_bad_arguments_before_touching_the_device():
    L = swz.lib
    p = swz.SwzParams(0, 0, 0, 0, 8)
    ref = ctypes.byref(p)
    A, B, C = 0x1000, 0x2000, 0x3000      # never dereferenced: every call below fails validation first
    assert L.swz_gemm_ex(None, B, C, 64, 64, 64, 0, 0, ref, None) == -1
    assert L.swz_gemm_ex(A, B, None, 64, 64, 64, 0, 0, ref, None) == -1
    assert L.swz_gemm_ex(A, B, C, 0, 64, 64, 0, 0, ref, None) == -1
    assert L.swz_gemm_ex(A, B, C, 64, 64, 64, 0, 8, ref, None) == -1
    assert L.swz_gemm_ex(A, B, C, 64, 64, 64, 1, 0, ref, None) == -2          # dtype
    assert L.swz_gemm_ex(A, B, C, 64, 64, 60, 0, 0, ref, None) == -2          # K % 8
    assert L.swz_gemm_ex(A, B, C, 64, 60, 64, 0, 0, ref, None) == -2          # N % 8
    assert L.swz_gemm_ex(A + 2, B, C, 64, 64, 64, 0, 0, ref, None) == -2      # alignment
    assert L.swz_gemm_ex(A, B, C, 1 << 31, 64, 64, 0, 0, ref, None) == -3


def test_persistent_closed_form_equals_constructive_oracle():
    for gm in range(1, 9):
        for gn in range(1, 9):
            for X in (1, 3, 4, 8):
                for G in (1, 2, 5, 8, 12, 64):
                    for mode in range(8):
                        got = swz.pid_map_persistent(gm, gn, X, 3, mode, G).tolist()
                        assert got == opm.pid_map_persistent(gm, gn, X, 3, mode, G), (gm, gn, X, G, mode)
    for gm, gn in [(16, 16), (32, 32), (64, 8), (40, 28), (79, 55)]:
        for mode in range(8):
            assert swz.pid_map_persistent(gm, gn, 8, 4, mode, 256).tolist() == opm.pid_map_persistent(gm, gn, 8, 4, mode, 256)


def test_persistent_error_paths():
    L = swz.lib
    out = np.full(64, -7, dtype=np.int32)
    assert L.swz_pid_map_persistent(4, 4, 8, 4, 0, 0, out.ctypes.data) == -1
    assert L.swz_pid_map_persistent(4, 4, 8, 4, 0, -3, out.ctypes.data) == -1
    assert L.swz_pid_map_persistent(4, 4, 8, 4, 8, 8, out.ctypes.data) == -1
    assert L.swz_pid_map_persistent(4, 4, 8, 4, 0, 8, None) == -1
    assert (out == -7).all()
    p = swz.gemm_plan(8192, 8192, 8192, num_xcd=8, persistent=1, num_wg=256)
    assert (p["persistent"], p["num_wg"]) == (1, 256)
    p = swz.gemm_plan(512, 512, 512, num_xcd=8, persistent=1, num_wg=256)
    assert p["num_wg"] == 16                                   # never more workgroups than tiles
    p = swz.gemm_plan(512, 512, 512, num_xcd=8)
    assert (p["persistent"], p["num_wg"]) == (0, 0)
    with pytest.raises(swz.SwzError):
        swz.gemm_plan(512, 512, 512, num_xcd=8, persistent=2)


def test_build_script_runs_without_importing_the_package():
    # the package refuses to import without libswz.so, so the build entry must not depend on importing it
    import importlib.util
    path = os.path.join(ROOT, "paper_2508_20258_amd", "build.py")
    spec = importlib.util.spec_from_file_location("swz_build_under_test", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    assert mod.build(force=False) == swz.binding.LIB_PATH          # up to date: returns without compiling
    entry = open(os.path.join(ROOT, "__graft_entry__.py")).read()
    assert "from paper_2508_20258_amd.build import" not in entry


def test_binding_refuses_tensors_of_another_device(monkeypatch):
    # the library launches on the current device; a tensor living elsewhere must be caught before the call
    import types

    import torch
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    here = types.SimpleNamespace(device=types.SimpleNamespace(index=0))
    there = types.SimpleNamespace(device=types.SimpleNamespace(index=1))
    swz.binding._same_current_device(None, here, here)
    with pytest.raises(ValueError):
        swz.binding._same_current_device(None, here, there)
    with pytest.raises(ValueError):
        swz.binding._same_current_device(there, here)
    swz.binding._same_current_device(here, here)


def test_launch_stream_takes_the_fast_way_only_on_the_current_device(monkeypatch):
    import types

    import torch
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d, raising=False)
    here, there = (types.SimpleNamespace(device=types.SimpleNamespace(index=i), get_device=lambda i=i: i) for i in (0, 1))
    stream = types.SimpleNamespace(device=types.SimpleNamespace(index=0), cuda_stream=77)
    away = types.SimpleNamespace(device=types.SimpleNamespace(index=1), cuda_stream=78)
    assert swz.binding._launch_stream(None, here, here) == 1000
    assert swz.binding._launch_stream(stream, here, here) == 77
    for bad in ((None, here, there), (stream, there), (away, here)):
        with pytest.raises(ValueError):
            swz.binding._launch_stream(*bad)


# few rows, long K: sub-tiles first, then workgroups that fetch ahead for them and compute nothing
@pytest.mark.parametrize("M,N,K,fed", [(1, 8, 2048, True), (32, 8192, 8192, True), (33, 4104, 2056, True), (128, 1000, 2048, True), (192, 64, 4096, True),
                                       (193, 1000, 8192, False), (192, 1000, 4088, False), (32, 8192, 2040, False), (32, 16384, 8192, False)])
def test_launch_map_of_fed_subtiles(M, N, K, fed):
    for mode, params in [(2, dict(num_xcd=8)), (0, dict(num_xcd=8)), (1, dict(num_xcd=3)), (3, dict(num_xcd=8, group_m=1)), (6, dict(num_xcd=8, group_m=1)),
                         (2, dict(num_xcd=1)), (2, dict(num_xcd=255)), (2, dict(num_xcd=1000))]:
        blocks = swz.gemm_launch_map(M, N, K, mode, **params)
        assert covers_once(blocks, M, N), (mode, params)
        computes = blocks[:, 2] > 0
        if mode == 2 and params["num_xcd"] == 8:
            assert fed == (len(blocks) == 256 and not computes.all())
        if not computes.all():
            assert len(blocks) == 256 and computes[:computes.sum()].all() and 16 * computes.sum() <= 9 * 256


def test_fast_call_leaves_what_is_not_ordinary_to_the_general_path():
    # without a GPU (or with tensors elsewhere, other types, non-integers) the fast call answers None and the general path says what is wrong
    torch = pytest.importorskip("torch")
    from paper_2508_20258_amd import binding
    x = torch.zeros((16, 16), dtype=torch.bfloat16)
    row = torch.zeros((16,), dtype=torch.bfloat16)
    fast = binding._fast
    for args in [(x, x, x, 2), (x, x, None, 2), (x, x, x, 2.0), (x, x, x, 1 << 40), (x, x, x), (3, x, x, 2), (x.t(), x, x, 2)]:
        assert fast.gemm(*args) is None
    assert fast.transpose(x, x, 64, 6) is None and fast.softmax(x, x, 1, 1) is None and fast.softmax(x, x, None, 1) is None
    assert fast.layernorm(x, row, row, x, 1e-5, 1, 1) is None and fast.layernorm(x, row, row, x, 0, 1, 1) is None and fast.layernorm() is None
    for call in (lambda: swz.gemm(x, x, x), lambda: swz.transpose(x, x), lambda: swz.softmax(x, x), lambda: swz.layernorm(x, row, row, x)):
        with pytest.raises(AssertionError):
            call()
    with pytest.raises(TypeError):
        fast.bind(1, 2)


def test_calls_without_an_output_do_not_try_the_fast_call(monkeypatch):
    # it would answer None to them: the general path makes the output
    torch = pytest.importorskip("torch")
    from paper_2508_20258_amd import binding
    tried = []

    class Recorder:
        def __getattr__(self, name):
            return lambda *args: tried.append(name)

    monkeypatch.setattr(binding, "_fast", Recorder())
    x = torch.zeros((16, 16), dtype=torch.bfloat16)
    row = torch.zeros((16,), dtype=torch.bfloat16)
    for call in (lambda **kw: swz.gemm(x, x, **kw), lambda **kw: swz.transpose(x, **kw), lambda **kw: swz.softmax(x, **kw), lambda **kw: swz.layernorm(x, row, row, **kw)):
        for kw in ({}, {"stream": object()}, {"num_xcd": 8}):
            with pytest.raises(AssertionError):
                call(**kw)
    assert not tried
    for call in (lambda: swz.gemm(x, x, x), lambda: swz.transpose(x, x), lambda: swz.softmax(x, x), lambda: swz.layernorm(x, row, row, x)):
        with pytest.raises(AssertionError):
            call()
    assert tried == ["gemm", "transpose", "softmax", "layernorm"]


def _build_module():
    import importlib.util
    spec = importlib.util.spec_from_file_location("swz_build_under_test", os.path.join(ROOT, "paper_2508_20258_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_build_finds_the_hip_headers_where_hipcc_is_a_bare_name(monkeypatch):
    mod = _build_module()
    for hipcc in ("hipcc", "/opt/rocm/bin/hipcc", "no-such-hipcc"):
        monkeypatch.setattr(mod, "HIPCC", hipcc)
        monkeypatch.setenv("PATH", "/opt/rocm/bin:" + os.environ["PATH"])
        assert os.path.exists(os.path.join(mod.rocm_include(), "hip", "hip_runtime.h")), hipcc


def test_build_makes_the_library_where_the_fast_call_does_not_build(monkeypatch, tmp_path):
    torch = pytest.importorskip("torch")
    mod = _build_module()
    monkeypatch.setattr(mod, "FAST", str(tmp_path / "_fastcall.so"))
    (tmp_path / "_fastcall.so").write_bytes(b"of another torch")
    made = []
    monkeypatch.setattr(mod, "build_lib", lambda *a, **k: made.append(a) or mod.LIB)
    for cxx in ("/nonexistent/g++", "false"):
        monkeypatch.setenv("CXX", cxx)
        with pytest.warns(RuntimeWarning, match="not built"):
            assert mod.build() == mod.LIB
        assert not os.path.exists(mod.FAST)                       # nothing stale is left to be loaded
    assert len(made) == 2
    monkeypatch.setattr(torch.version, "hip", None)               # a torch without ROCm: nothing to build, nothing to warn of
    assert mod.build() == mod.LIB and mod.build_fastcall() is None


def test_fast_call_is_built_again_for_another_torch_or_header(monkeypatch, tmp_path):
    torch = pytest.importorskip("torch")
    mod = _build_module()
    header = tmp_path / "swz.h"
    header.write_text("")
    os.utime(header, (os.path.getmtime(mod.FAST) - 10,) * 2)
    assert any(os.path.samefile(d, os.path.join(ROOT, "include", "swz.h")) for d in mod.FAST_DEPS)
    monkeypatch.setattr(mod, "FAST_DEPS", [str(header)])
    assert mod.fastcall_is_current(torch)
    os.utime(header, (os.path.getmtime(mod.FAST) + 10,) * 2)
    assert not mod.fastcall_is_current(torch)
    os.utime(header, (os.path.getmtime(mod.FAST) - 10,) * 2)
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".1")
    assert not mod.fastcall_is_current(torch)


@pytest.mark.parametrize("how", ["missing", "another torch", "torch without ROCm"])
def test_package_works_without_the_fast_call(how):
    import subprocess
    import sys
    pytest.importorskip("torch")
    code = f"""
import sys, types, warnings
import torch
how = {how!r}
if how == "missing":
    sys.modules["paper_2508_20258_amd._fastcall"] = None
elif how == "another torch":
    sys.modules["paper_2508_20258_amd._fastcall"] = types.SimpleNamespace(built_for="swz built for torch 1.0")
else:
    torch.version.hip = None
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    import paper_2508_20258_amd as swz
assert [x.category for x in w if "_fastcall" in str(x.message)] == ([] if how == "torch without ROCm" else [RuntimeWarning]), w
assert swz.pid_map(4, 5, 4, 4, 1).tolist()[0] == 0 and swz.gemm_plan(512, 512, 512, num_xcd=8)["bm"] == 128
x = torch.zeros((16, 16), dtype=torch.bfloat16)
for call in (lambda: swz.gemm(x, x, x), lambda: swz.transpose(x, x), lambda: swz.softmax(x, x), lambda: swz.layernorm(x, x[0], x[0], x)):
    try:
        call()
    except AssertionError:
        continue
    raise SystemExit("not the general path")
"""
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


def test_no_sub_tile_reads_beyond_its_source_offsets():
    # (rows - 1) * K * 2 fits 32 bits for every block of a launch
    for K in (1 << 22, (1 << 23) - 8, 1 << 23, 11184816, (1 << 24) - 8):
        for M, N in [(1537, 2680), (4575, 1112), (193, 12304), (577, 3848)]:
            rows = int(swz.gemm_launch_map(M, N, K, 2, num_xcd=8)[:, 2].max())
            assert rows * K * 2 < 1 << 32, (M, N, K, rows)


# a third and a fourth row of sub-tiles, each of which reads all of B, and a K of one stage: 128 rows; else 96
@pytest.mark.parametrize("M,N,K,rows", [(203, 9576, 264, 128), (193, 10400, 2056, 128), (239, 9000, 2056, 128), (240, 9000, 504, 128), (240, 9000, 520, 96),
                                        (256, 9000, 2056, 96), (289, 6792, 168, 128), (300, 6792, 320, 128), (300, 6792, 328, 96), (384, 6792, 520, 96),
                                        (440, 5200, 64, 128), (440, 5200, 72, 96), (170, 11504, 256, 96), (170, 11504, 64, 128), (274, 9008, 72, 96)])
def test_sub_tiles_of_96_rows(M, N, K, rows):
    blocks = swz.gemm_launch_map(M, N, K, 2, num_xcd=8)
    assert tuple(blocks[:, 2:].max(axis=0)) == (rows, 128)
