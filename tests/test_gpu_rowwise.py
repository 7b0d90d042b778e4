"""GPU parity of the row softmax / layer normalisation entry points (through the C ABI) against the fp64 oracle."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import rowwise_ref as rw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NEG_INF = np.uint16(0xFF80)          # bfloat16 -inf


@pytest.fixture(scope="module")
def swz():
    import paper_2508_20258_amd as m
    assert torch.cuda.is_available()
    return m


def to_dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def to_bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


SHAPES = [(1, 8, 1), (3, 40, 5), (17, 1000, 1), (17, 1000, 3), (17, 1000, 8), (64, 4096, 8), (5, 72, 4),
          (9, 8200, 7), (2, 262144, 16), (300, 2048, 2), (1031, 264, 3),
          # one workgroup per row: a row per wave (N <= 2048), rows kept in registers (N <= 32768), rows streamed twice
          (7, 2048, 1), (65, 1000, 1), (33, 2056, 1), (12, 8192, 1), (5, 32768, 1), (3, 32776, 1), (2, 100000, 1)]


def run_all_modes(fn, M, N):
    outs = []
    for mode in range(4):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        fn(out, mode)
        torch.cuda.synchronize()
        outs.append(to_bits(out))
    for o in outs[1:]:
        assert np.array_equal(o, outs[0]), "result bits depend on the mode"
    return outs[0]


@pytest.mark.parametrize("M,N,chunks", SHAPES)
@pytest.mark.parametrize("scale", [1.0, 6.0])
def test_softmax_matches_oracle_in_every_mode(swz, M, N, chunks, scale):
    x = si.matrix_bf16(700 + N, 0, M, N, "normal", scale)
    if N >= 40:
        x[0, 3:N:7] = NEG_INF                       # masked entries
        x[M - 1, :N - 1] = NEG_INF                  # a row with a single finite entry
    xd = to_dev(x)
    got = run_all_modes(lambda out, mode: swz.softmax(xd, out, chunks=chunks, mode=mode), M, N)
    ref = rw.softmax(x)
    err = np.abs(si.bf16_bits_to_f64(got) - ref)
    ok = err <= rw.softmax_bound(ref)
    assert ok.all(), f"{np.count_nonzero(~ok)} of {ok.size} outside tolerance, worst {err.max()}"
    # the result does not depend on num_xcd / group_m, nor (with 256 threads per row) on how the row is cut
    one = swz.softmax(xd, chunks=1, mode=0)
    odd = swz.softmax(xd, chunks=chunks, mode=2, num_xcd=3, group_m=7)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(odd), got)
    if N > 2048:
        assert np.array_equal(to_bits(one), got)
    else:
        assert (np.abs(si.bf16_bits_to_f64(to_bits(one)) - ref) <= rw.softmax_bound(ref)).all()


@pytest.mark.parametrize("M,N,chunks", SHAPES)
@pytest.mark.parametrize("offset", [0.0, 200.0])
def test_layernorm_matches_oracle_in_every_mode(swz, M, N, chunks, offset):
    eps = 1e-5
    x = si.f32_to_bf16_bits((si.bf16_bits_to_f64(si.matrix_bf16(800 + N, 0, M, N, "normal", 2.0)) + offset).astype(np.float32))
    g = si.matrix_bf16(800 + N, 1, 1, N, "uniform", 2.0)[0]
    b = si.matrix_bf16(800 + N, 2, 1, N, "uniform")[0]
    xd, gd, bd = to_dev(x), to_dev(g), to_dev(b)
    got = run_all_modes(lambda out, mode: swz.layernorm(xd, gd, bd, out, eps=eps, chunks=chunks, mode=mode), M, N)
    ref = rw.layernorm(x, g, b, eps)
    err = np.abs(si.bf16_bits_to_f64(got) - ref)
    ok = err <= rw.layernorm_bound(x, g, b, eps)
    assert ok.all(), f"{np.count_nonzero(~ok)} of {ok.size} outside tolerance, worst {err.max()}"
    one = swz.layernorm(xd, gd, bd, eps=eps, chunks=1, mode=0)
    odd = swz.layernorm(xd, gd, bd, eps=eps, chunks=chunks, mode=2, num_xcd=3, group_m=7)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(odd), got)
    if N > 2048:
        assert np.array_equal(to_bits(one), got)
    else:
        assert (np.abs(si.bf16_bits_to_f64(to_bits(one)) - ref) <= rw.layernorm_bound(x, g, b, eps)).all()


def test_layernorm_constant_and_exact_rows(swz):
    # a constant row has variance 0: y = beta; rows of +-1 with gamma = 1, beta = 0, eps = 0 come back unchanged
    N = 512
    x = np.empty((2, N), dtype=np.float32)
    x[0] = 3.0
    x[1] = np.where(np.arange(N) % 2 == 0, -1.0, 1.0)
    xd = to_dev(si.f32_to_bf16_bits(x))
    g = torch.ones(N, dtype=torch.bfloat16, device="cuda")
    b = torch.full((N,), 0.5, dtype=torch.bfloat16, device="cuda")
    y = swz.layernorm(xd, g, b, eps=1e-5, chunks=2, mode=1).float().cpu().numpy()
    assert (y[0] == 0.5).all()
    y = swz.layernorm(xd, g, torch.zeros_like(b), eps=0.0, chunks=2, mode=1).float().cpu().numpy()
    assert np.array_equal(y[1], x[1])


def test_rowwise_full_size_in_the_measured_configuration(swz):
    # the shape and launch the profiling harness times: 8192 x 8192, 8 chunks per row; oracle on sampled rows
    M = N = 8192
    x = si.matrix_bf16(31, 0, M, N, "normal", 2.0)
    g = si.matrix_bf16(31, 1, 1, N, "uniform", 2.0)[0]
    b = si.matrix_bf16(31, 2, 1, N, "uniform")[0]
    xd, gd, bd = to_dev(x), to_dev(g), to_dev(b)
    rows = np.unique(np.concatenate([[0, 1, 7, 8, M - 1], (np.arange(64) * 2654435761 % M)]))
    sm = {mode: to_bits(swz.softmax(xd, chunks=8, mode=mode)) for mode in (0, 1)}
    ln = {mode: to_bits(swz.layernorm(xd, gd, bd, eps=1e-5, chunks=8, mode=mode)) for mode in (0, 1)}
    torch.cuda.synchronize()
    assert np.array_equal(sm[0], sm[1]) and np.array_equal(ln[0], ln[1])
    ref = rw.softmax(x[rows])
    assert (np.abs(si.bf16_bits_to_f64(sm[1][rows]) - ref) <= rw.softmax_bound(ref)).all()
    ref = rw.layernorm(x[rows], g, b, 1e-5)
    assert (np.abs(si.bf16_bits_to_f64(ln[1][rows]) - ref) <= rw.layernorm_bound(x[rows], g, b, 1e-5)).all()
    # properties that hold for every row: probabilities sum to 1 within the output rounding
    sums = si.bf16_bits_to_f64(sm[1]).sum(axis=1)
    assert np.abs(sums - 1.0).max() < 2e-3


def test_rowwise_error_paths(swz):
    x = to_dev(si.matrix_bf16(1, 0, 16, 64, "uniform"))
    y = torch.full((16, 64), 2.0, dtype=torch.bfloat16, device="cuda")
    g = torch.ones(64, dtype=torch.bfloat16, device="cuda")
    L = swz.lib
    s = torch.cuda.current_stream().cuda_stream
    xp, yp, gp = x.data_ptr(), y.data_ptr(), g.data_ptr()
    assert L.swz_softmax(xp, yp, 16, 64, 0, 0, None, s) == -1          # chunks < 1
    assert L.swz_softmax(xp, yp, 16, 64, 9, 0, None, s) == -1          # more chunks than 16-byte vectors
    assert L.swz_softmax(xp, yp, 16, 60, 1, 0, None, s) == -2          # N % 8
    assert L.swz_softmax(xp, yp, 16, 64, 1, 8, None, s) == -1          # mode
    assert L.swz_softmax(xp, yp, 16, 64, 1, 5, None, s) == -2          # skewed modes would pull a row's chunks apart: not offered
    assert L.swz_layernorm(xp, gp, gp, yp, 16, 64, 1e-5, 1, 6, None, s) == -2
    assert L.swz_softmax(None, yp, 16, 64, 1, 0, None, s) == -1
    assert L.swz_softmax(xp + 2, yp, 16, 56, 1, 0, None, s) == -2      # alignment
    assert L.swz_softmax(xp, yp, 1 << 28, 64, 8, 0, None, s) == -3     # M * chunks
    assert L.swz_layernorm(xp, None, gp, yp, 16, 64, 1e-5, 1, 0, None, s) == -1
    assert L.swz_layernorm(xp, gp, gp, yp, 16, 64, -1.0, 1, 0, None, s) == -1
    assert L.swz_layernorm(xp, gp, gp, yp, 16, 64, float("nan"), 1, 0, None, s) == -1
    assert L.swz_layernorm(xp, gp, gp, yp, 16, 1 << 25, 1e-5, 1, 0, None, s) == -2
    torch.cuda.synchronize()
    assert (y == 2.0).all()


# Every way a row is held: the last N of each shape and the first of the next (16 to 64 lanes, 256 to 1024 threads), and the two
# launches above 98304 elements (ragged segments and chunks; M chosen so that the last group of rows is ragged too)
ROW_EDGES = [(33, 8), (33, 128), (17, 136), (17, 256), (9, 264), (9, 512), (9, 520), (5, 1024), (5, 1032), (6, 1792), (3, 1800),
             (3, 4096), (3, 4104), (2, 8200), (2, 12288), (2, 12296), (2, 16384), (2, 16392), (3, 32776), (2, 40960), (2, 40968),
             (2, 49160), (2, 65536), (2, 65544), (1, 81920), (2, 81928), (2, 98304), (3, 98312), (2, 131080), (1, 1 << 20), (1, 3145736)]


@pytest.mark.parametrize("M,N", ROW_EDGES)
def test_every_row_shape_matches_oracle(swz, M, N):
    x = si.matrix_bf16(900 + M, 0, M, N, "normal", 3.0)
    g, b = si.matrix_bf16(900 + M, 1, 1, N, "uniform", 2.0)[0], si.matrix_bf16(900 + M, 2, 1, N, "uniform")[0]
    xs = x.copy()
    xs[0, 1::3] = NEG_INF                           # masked entries; in the last row everything but its end, so that
    xs[M - 1, :N - 5] = NEG_INF                     # whole vectors, lanes and segments hold nothing else
    xd, xsd, gd, bd = to_dev(x), to_dev(xs), to_dev(g), to_dev(b)
    chunks = min(8, N // 8)
    out = torch.full((M + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    got = run_all_modes(lambda o, mode: swz.softmax(xsd, o, chunks=chunks, mode=mode), M, N)
    swz.softmax(xsd, out[:M], chunks=1, mode=1, num_xcd=3)
    assert np.array_equal(to_bits(out[:M]), got) and torch.isnan(out[M]).all()
    ref = rw.softmax(xs)
    assert (np.abs(si.bf16_bits_to_f64(got) - ref) <= rw.softmax_bound(ref)).all()
    got = run_all_modes(lambda o, mode: swz.layernorm(xd, gd, bd, o, eps=1e-5, chunks=chunks, mode=mode), M, N)
    swz.layernorm(xd, gd, bd, out[:M], eps=1e-5, chunks=1, mode=1, num_xcd=3)
    assert np.array_equal(to_bits(out[:M]), got) and torch.isnan(out[M]).all()
    ref = rw.layernorm(x, g, b, 1e-5)
    assert (np.abs(si.bf16_bits_to_f64(got) - ref) <= rw.layernorm_bound(x, g, b, 1e-5)).all()


@pytest.mark.parametrize("N", [64, 200, 1000, 5000, 40000, 200000])
def test_softmax_of_infinities_nan_and_extreme_rows(swz, N):
    x = torch.randn((5, N), device="cuda").to(torch.bfloat16)
    x[0] = float("-inf")                            # no finite entry: NaN
    x[1, N // 2] = float("nan")
    x[2, N - 1] = float("inf")
    x[3] = -3.0e38                                  # equal finite entries, however large: 1 / N
    y = swz.softmax(x).float()
    assert torch.isnan(y[:3]).all()
    assert (y[3] == torch.tensor(1.0 / N, dtype=torch.float64).to(torch.bfloat16).item()).all()
    assert abs(y[4].double().sum().item() - 1.0) < 4e-3     # the row between them is untouched: half an ulp a value


# One N per way a row is held: 16, 32, 64 lanes, a workgroup with one and with several vectors a thread, two launches
FORMS = [64, 200, 1000, 1800, 5000, 12304, 40000, 98312, 200000]


@pytest.mark.parametrize("N", FORMS)
def test_softmax_of_rows_of_large_magnitude(swz, N):
    # exp(x - max) of the largest entry is 1 whatever its size; 2^20 and 255 * 2^12 are neighbours among bfloat16 numbers
    top = float(2 ** 20)
    flat = [3e9, -1e10, 1e30, -1e30, 3e38, -3e38, float(torch.finfo(torch.bfloat16).min), top, -top, 1e6, -1e6, 12345.0]
    rows = torch.empty((len(flat) + 6, N))
    for i, v in enumerate(flat):
        rows[i] = v                                         # equal entries: 1 / N
    g = torch.Generator().manual_seed(N)
    rows[len(flat):] = torch.randn((6, N), generator=g) * 3
    rows[-6, N // 3] = 1e10                                 # one entry, and one of two, far above the others
    rows[-5, N // 5], rows[-5, N - 1] = 1e30, 1e30
    rows[-4, : N // 2] = -1e30                              # masks of large finite values
    rows[-3, 1:] = float(torch.finfo(torch.bfloat16).min)
    rows[-2, : N // 2], rows[-2, N // 2:] = top, top - 4096
    rows[-1, : N // 2], rows[-1, N // 2:] = -top, 4096 - top
    x = rows.to(torch.bfloat16)
    got = run_all_modes(lambda out, mode: swz.softmax(x.cuda(), out, chunks=min(3, N // 8), mode=mode), x.shape[0], N)
    ref = rw.softmax(to_bits(x))
    err = np.abs(si.bf16_bits_to_f64(got) - ref)
    bad = ~(err <= rw.softmax_bound(ref)).all(axis=1)
    assert not bad.any(), f"rows {np.nonzero(bad)[0].tolist()} of N = {N}"


@pytest.mark.parametrize("N", FORMS + [16384, 65544, 98304, 131080, 250000, 500000, 1000000, 3145736])
def test_layernorm_of_constant_rows_is_beta(swz, N):
    # a sum of N equal bfloat16 numbers is exact (N is a multiple of 8 of at most 14 more bits, or cut into segments that are),
    # so the mean is the number itself, the deviations are 0 and not one ulp of the mean times 1 / sqrt(eps)
    values = [3.0, -0.37109375, 100.0, 1000.0, -10048.0, 1e6, 3e9, -1e15]
    x = torch.tensor(values).to(torch.bfloat16)[:, None].expand(-1, N).contiguous().cuda()
    g = torch.randn(N, device="cuda").to(torch.bfloat16)
    b = torch.randn(N, device="cuda").to(torch.bfloat16)
    y = swz.layernorm(x, g, b)
    torch.cuda.synchronize()
    assert torch.equal(y, b.expand_as(y))


@pytest.mark.parametrize("N", FORMS)
def test_layernorm_of_rows_whose_sum_is_beyond_fp32(swz, N):
    # eight entries still have a sum in fp32, the row has not; y = beta where they are equal
    values = torch.tensor([1e35, -1e37, 4e37, -4e37]).to(torch.bfloat16)
    x = values[:, None].expand(-1, N).contiguous().cuda()
    g = torch.randn(N, device="cuda").to(torch.bfloat16)
    b = torch.randn(N, device="cuda").to(torch.bfloat16)
    y = swz.layernorm(x, g, b)
    x[0] = (1e35 * (1 + torch.rand(N, device="cuda"))).to(torch.bfloat16)       # squared deviations beyond fp32 too
    z = swz.layernorm(x, g, b)
    torch.cuda.synchronize()
    assert torch.equal(y, b.expand_as(y))
    assert torch.isfinite(z).all()


@pytest.mark.parametrize("op,M,N", [("softmax", (1 << 28) + 5, 8), ("layernorm", (1 << 28) + 5, 8), ("softmax", (1 << 24) + 3, 1800),
                                    ("layernorm", (1 << 24) + 3, 1800), ("softmax", (1 << 23) + 3, 4104)])
def test_more_rows_than_a_launch_has_threads_for(swz, op, M, N):
    # rows x threads a row pass 2^32; every row repeats one of `block`, whose results a small launch gives
    block = (torch.randn((4096, N), device="cuda") * 2).to(torch.bfloat16)
    g, b = torch.randn((2, N), device="cuda").to(torch.bfloat16)
    call = (lambda t: swz.softmax(t)) if op == "softmax" else (lambda t: swz.layernorm(t, g, b))
    want = call(block)
    y = call(block.repeat(-(-M // 4096), 1)[:M])
    whole = y[:M // 4096 * 4096].view(-1, 4096, N)
    step = max(1, (1 << 31) // (4096 * N))
    for i in range(0, whole.shape[0], step):
        assert (whole[i:i + step].view(torch.int16) == want.view(torch.int16)).all(), i
    assert torch.equal(y[M // 4096 * 4096:], want[:M % 4096])
    del y, whole
    torch.cuda.empty_cache()                        # up to 140 GB


# more rows than compute units: two long rows to a compute unit (softmax from 40968 to 65536 elements and up to 8 or 16 rows to each, layer normalisation from
# 32776 to 49152), row after row (layer normalisation to 8192, one and two workgroups to each).  The bits are those of the same rows in calls with few.
@pytest.mark.parametrize("op,M,N", [("softmax", 258, 40968), ("softmax", 300, 49152), ("softmax", 257, 49160), ("softmax", 261, 65536), ("softmax", 4096, 41000), ("softmax", 2049, 49160),
                                    ("layernorm", 258, 32776), ("layernorm", 300, 40960), ("layernorm", 257, 40968), ("layernorm", 261, 49152),
                                    ("layernorm", 513, 6000), ("layernorm", 1100, 8192), ("layernorm", 4800, 7008), ("layernorm", 1025, 3400),
                                    ("layernorm", 1537, 4096), ("layernorm", 513, 8192),
                                    ("layernorm", 1409, 3600), ("layernorm", 1408, 3600), ("layernorm", 1537, 3592), ("layernorm", 1536, 3400)])
def test_many_rows_give_the_bits_of_few(swz, op, M, N):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = (torch.randn((M, N), device="cuda", generator=g) * 2 + 0.5).to(torch.bfloat16)
    gamma, beta = (torch.randn((N,), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    if op == "softmax":
        x[M // 2] = float("-inf")
        x[M - 1, N - 1] = 3e38
        x[0, 0] = float("nan")

    def call(rows, out):
        return swz.softmax(rows, out) if op == "softmax" else swz.layernorm(rows, gamma, beta, out)

    buf = torch.full((M + 2, N), 7.0, dtype=torch.bfloat16, device="cuda")
    call(x, buf[1:M + 1])
    torch.cuda.synchronize()
    assert (buf[0] == 7).all() and (buf[M + 1] == 7).all()
    for r in range(0, M, 250):
        want = call(x[r:r + 250], torch.empty_like(x[r:r + 250]))
        assert torch.equal(buf[1 + r:1 + r + len(want)].view(torch.int16), want.view(torch.int16)), r
    inplace = x.clone()
    call(inplace, inplace)
    assert torch.equal(inplace.view(torch.int16), buf[1:M + 1].view(torch.int16))


# the maximum of a row: rows of negative numbers only, zeros of both signs, infinities and NaNs of both signs, every place in a vector
@pytest.mark.parametrize("N", [64, 264, 2048, 33000, 49152])
def test_softmax_maximum_of_every_sign(swz, N):
    g = torch.Generator(device="cuda").manual_seed(N)
    base = -(torch.rand((40, N), device="cuda", generator=g) * 60 + 1)
    rows = base.clone()
    for r in range(8):
        rows[r, (N // 8 // 2) * 8 + r] = -0.5                       # the largest of a negative row
        rows[8 + r, N - 8 + r] = -0.0
        rows[16 + r, r] = 30.0
        rows[24 + r, r] = float("-inf")
    rows[32, 3], rows[33, 4] = float("inf"), float("nan")
    rows[34] = float("-inf")
    rows[35] = -0.0
    rows[36, 1] = 0.0
    rows[36, 2] = -0.0
    x = rows.to(torch.bfloat16)
    bits = x.view(torch.int16)
    bits[37, 6] = -64                                               # 0xFFC0, a NaN with its sign set
    bits[38, :] = -64
    x = x.repeat(8, 1)                                              # more rows than compute units
    y = swz.softmax(x).double().cpu()
    want = torch.softmax(x.double(), dim=1).cpu()
    assert torch.equal(torch.isnan(y), torch.isnan(want))
    ok = ~torch.isnan(want)
    assert ((y - want).abs()[ok] <= 2.0 ** -8 * want[ok] + 1e-30).all()
