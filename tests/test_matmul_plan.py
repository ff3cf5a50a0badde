"""Host tests of the dispatch of the plain matmuls (relax_plan_matmul): which kernel, k cut and tile sizes take."""
import pytest

from paper_2311_02103_amd import binding as rx


def plan(fmt, n, m, k, ws_bytes=0, group=32):
    rc, *rest = rx.relax_plan_matmul(fmt, n, m, k, ws_bytes, group)
    assert rc == rx.OK
    return tuple(rest)


def workspace(n, m, k):
    """What relax_matmul_workspace_bytes gives for a 4-bit matrix (any pointers do)."""
    return rx.relax_matmul_workspace_bytes(rx.QMat(256, 256, m, k, 32), n)


def test_errors():
    assert rx.relax_plan_matmul("q5", 1, 64, 64)[0] == rx.ERR_UNSUPPORTED
    for n, m, k in ((0, 64, 64), (1, 0, 64), (1, 64, 0), (1, 64, 40)):
        assert rx.relax_plan_matmul("q4", n, m, k)[0] == rx.ERR_SHAPE
    for fmt, group in (("q4", 48), ("q4", 256), ("q3", 64), ("f16", 128)):
        assert rx.relax_plan_matmul(fmt, 8, 256, 256, 0, group)[0] == rx.ERR_UNSUPPORTED


@pytest.mark.parametrize("fmt", ["q4", "q3", "f16"])
def test_the_dispatch_follows_the_row_count(fmt):
    m, k = 4096, 4096
    ws = workspace(128, m, k) if fmt == "q4" else 0
    kernels = [plan(fmt, n, m, k, ws)[0] for n in (1, 8, 300)]
    assert kernels == [rx.KERNEL_MATVEC, rx.KERNEL_STREAM, rx.KERNEL_TILED]
    assert plan(fmt, 300, 250, 1000 // 32 * 32, ws)[0] == rx.KERNEL_MATVEC         # m % 4, k % 128: no MFMA kernel takes it
    assert plan("q4", 8, m, k, 0)[0] == rx.KERNEL_MATVEC                          # the few-row kernels need the workspace


def test_a_launch_cut_along_k_stays_within_its_workspace():
    for n, m, k in ((129, 4096, 4096), (300, 4096, 11008), (511, 8192, 28672)):
        full = workspace(n, m, k)
        for ws in (0, full // 3, full):
            kernel, ranges, *_ = plan("q4", n, m, k, ws)
            assert kernel == rx.KERNEL_TILED and (ranges == 1 or ranges * n * m * 4 <= ws)


# Measured times in us (weights cold, the best of several replays of a captured schedule): the streaming kernel at its best k cut and
# the split-K kernel, 4-bit weights in groups of 32.  Where they differ by more than a twentieth the dispatch has to find the faster one.
FEW_ROWS = [
    (2048, 2048, 16, 7.1, 11.1), (4096, 4096, 8, 8.4, 11.9), (12288, 4096, 8, 12.1, 14.9), (22016, 4096, 16, 19.1, 23.4),
    (22016, 4096, 64, 35.0, 38.0), (57344, 8192, 16, 58.5, 74.5), (57344, 8192, 32, 72.5, 88.9), (27648, 5120, 16, 25.0, 30.5),
    (4096, 11008, 24, 19.6, 17.0), (4096, 11008, 32, 20.6, 17.3), (5120, 13824, 8, 18.4, 16.9), (5120, 13824, 16, 20.0, 17.8),
    (5120, 13824, 32, 24.2, 19.9), (5120, 13824, 64, 31.2, 26.9), (8192, 8192, 16, 18.8, 16.5), (8192, 8192, 32, 23.0, 18.8),
    (8192, 8192, 64, 31.1, 25.5), (10240, 8192, 32, 25.1, 22.1), (15360, 5120, 32, 24.6, 22.4), (15360, 5120, 64, 35.8, 29.9),
    (5120, 13824, 2, 17.6, 15.9), (8192, 8192, 4, 16.7, 15.5), (7168, 7168, 32, 20.9, 18.1), (16384, 3072, 40, 25.4, 20.1), (32000, 2048, 48, 31.6, 24.8),
    (12288, 12288, 8, 25.4, 35.4), (30000, 1024, 15, 10.6, 12.4), (5120, 25600, 8, 24.7, 29.4), (2560, 10240, 5, 12.2, 13.9),
    (9216, 9216, 24, 25.2, 22.1), (36864, 4608, 40, 50.5, 61.2), (51200, 5120, 17, 47.2, 56.2), (11264, 2048, 48, 15.1, 17.8),
]


@pytest.mark.parametrize("m,k,n,stream,split", FEW_ROWS)
def test_few_rows_take_the_faster_kernel(m, k, n, stream, split):
    assert plan("q4", n, m, k, workspace(n, m, k))[0] == (rx.KERNEL_STREAM if stream < split else rx.KERNEL_SPLIT_K)


# The same for the calls without a workspace or an epilogue: the streaming kernel, and the matvec kernel or (from 16 rows of 3-bit
# weights on) the tiled GEMM that takes the call otherwise.
ALONE = [
    ("q3", 22016, 4096, 2, 19.2, 14.0), ("q3", 8192, 8192, 2, 16.5, 12.1), ("q3", 4096, 11008, 2, 13.3, 14.6), ("q3", 5632, 2048, 4, 7.7, 6.7),
    ("q3", 4096, 4096, 4, 8.0, 10.2), ("q3", 1024, 1024, 8, 5.2, 4.4), ("q3", 256, 768, 15, 5.2, 4.0), ("q3", 1024, 1024, 15, 5.4, 5.8),
    ("q3", 22016, 4096, 8, 19.6, 32.1), ("q3", 768, 256, 32, 5.7, 5.3), ("q3", 256, 768, 32, 6.3, 9.1), ("q3", 768, 256, 64, 7.2, 5.8),
    ("q3", 32000, 2048, 40, 28.8, 24.1), ("q3", 5632, 2048, 40, 12.4, 19.8),
    ("f16", 8192, 8192, 2, 32.6, 28.7), ("f16", 22016, 4096, 3, 34.8, 54.0), ("f16", 28672, 4096, 2, 41.5, 43.3), ("f16", 5120, 5120, 4, 17.2, 15.7),
    ("f16", 10240, 8192, 4, 37.0, 35.2), ("f16", 12288, 4096, 8, 20.5, 44.0), ("f16", 1024, 1024, 8, 5.9, 4.8), ("f16", 4096, 4096, 8, 11.4, 16.1),
    ("f16", 4096, 4096, 32, 15.5, 42.6),
]


@pytest.mark.parametrize("fmt,m,k,n,stream,other", ALONE)
def test_calls_without_a_workspace_take_the_faster_kernel(fmt, m, k, n, stream, other):
    assert (plan(fmt, n, m, k)[0] == rx.KERNEL_STREAM) == (stream < other)


# The tiled GEMM's tiles (weight rows, rows of x, k splits) with their measured times in us: the fastest ones, and the one that one
# figure per tile would pick.  The plan has to be within a tenth of the fastest.
TILES = [
    ("q4", 12288, 4096, 600, {(256, 128, 1): 64, (128, 128, 1): 70, (256, 192, 1): 79, (128, 192, 1): 97}),
    ("q4", 22016, 4096, 560, {(256, 128, 1): 120, (128, 128, 1): 128, (128, 192, 1): 145, (256, 192, 1): 154}),
    ("q4", 4096, 11008, 300, {(128, 192, 4): 46.9, (128, 64, 3): 47.3, (256, 128, 5): 47.7, (256, 192, 8): 47.9, (128, 128, 5): 50.6}),
    ("q4", 8192, 28672, 511, {(256, 256, 4): 205, (256, 128, 2): 215, (256, 256, 8): 222, (128, 256, 2): 227}),
    ("q4", 10240, 8192, 200, {(256, 128, 3): 54.1, (128, 256, 3): 54.7, (256, 256, 6): 57.4, (128, 128, 3): 58.1}),
    ("q3", 12288, 4096, 640, {(128, 128, 1): 86, (256, 192, 1): 97, (128, 192, 1): 117}),
    ("q3", 22016, 4096, 513, {(128, 128, 1): 152, (128, 192, 1): 174, (256, 192, 1): 181}),
    ("f16", 12288, 4096, 600, {(128, 128, 1): 96, (128, 192, 1): 112, (256, 192, 1): 118}),
    ("f16", 22016, 4096, 300, {(128, 192, 1): 117, (256, 192, 1): 126, (128, 256, 1): 133}),
    ("f16", 27648, 5120, 2048, {(128, 256, 1): 667, (256, 256, 1): 741, (128, 192, 1): 795, (256, 192, 1): 882}),
    ("f16", 32000, 4096, 700, {(128, 256, 1): 231, (128, 192, 1): 259, (256, 192, 1): 267}),
    ("f16", 15360, 5120, 1200, {(128, 256, 1): 260, (128, 128, 1): 293, (128, 192, 1): 298, (256, 192, 1): 302}),
]


@pytest.mark.parametrize("fmt,m,k,n,us", TILES)
def test_tile_plan_picks_a_fast_tile(fmt, m, k, n, us):
    kernel, splits, rows, cols, _ = plan(fmt, n, m, k, 8 * n * m * 4 if fmt == "q4" and n <= 512 else 0)
    assert kernel == rx.KERNEL_TILED
    assert us[rows, cols, splits] <= 1.1 * min(us.values())


# Two launches, whole rounds of 256 x 256 tiles first (us: two launches, the best single one): 4-bit only.
TWO_LAUNCHES = [(12288, 4096, 2048, 8192, 185, 194), (27648, 5120, 2048, 24576, 491, 515), (22016, 4096, 1700, 18432, 288, 310), (32000, 4096, 1700, 27648, 400, 415)]


@pytest.mark.parametrize("m,k,n,wide,us_two,us_one", TWO_LAUNCHES)
def test_tall_matrices_are_cut_into_two_launches(m, k, n, wide, us_two, us_one):
    assert us_two < us_one and plan("q4", n, m, k) == (rx.KERNEL_TILED, 1, 128, 256, wide)
    assert plan("q3", n, m, k)[4] == plan("f16", n, m, k)[4] == 0


# Tall matrices at up to 64 rows: the streaming kernel, the split-K kernel and the tiled GEMM in us.  The tiled GEMM is a candidate from 48 rows on.
TALL = [(57344, 8192, 47, None, None, None), (57344, 8192, 48, 99, 143, 87), (57344, 8192, 56, 102, 147, 88), (57344, 8192, 64, 105, 151, 90),
        (49152, 2048, 48, 45.3, 41.2, 26.5), (51200, 5120, 48, 67, 95, 56), (128256, 4096, 64, 117, 156, 97)]


@pytest.mark.parametrize("m,k,n,stream,split,tiled", TALL)
def test_tall_matrices_go_to_the_tiled_gemm_from_48_rows(m, k, n, stream, split, tiled):
    assert n < 48 or tiled < min(stream, split)
    assert plan("q4", n, m, k, workspace(n, m, k))[0] == (rx.KERNEL_STREAM if n < 48 else rx.KERNEL_TILED)


# Groups of 64 and 128 at 33 to 64 rows: the streaming kernel and the split-K kernel in us (groups of 128).
COARSE = [(22016, 4096, 33, 29.6, 36.0), (22016, 4096, 64, 34.7, 39.3), (27648, 5120, 33, 44.4, 49.0), (27648, 5120, 64, 46.4, 54.4), (57344, 8192, 33, 96, 136),
          (8192, 28672, 33, 56.5, 73.3), (8192, 28672, 64, 62.3, 79.3), (2048, 2048, 48, 10.8, 15.1), (4096, 4096, 33, 14.2, 16.6), (20, 5120, 33, 11.2, 13.4)]


@pytest.mark.parametrize("m,k,n,stream,split", COARSE)
@pytest.mark.parametrize("group", [64, 128])
def test_long_groups_stay_on_the_streaming_kernel_at_33_to_64_rows(group, m, k, n, stream, split):
    assert stream < split and plan("q4", n, m, k, workspace(n, m, k), group)[0] == rx.KERNEL_STREAM
    for rows in range(33, 65):                            # decoded alike: one route for all groups
        assert plan("q4", rows, m, k, workspace(rows, m, k), group) == plan("q4", rows, m, k, workspace(rows, m, k)), rows


# Rows of 10241 to 12288 columns in one k range are six units per wavefront: streaming kernel with them, without (two ranges or more) in us, groups of 32.
SIX_UNITS = [(4096, 11008, 2, 11.6, 12.8), (4096, 11008, 4, 12.5, 13.2), (4096, 11008, 6, 12.9, 14.4), (12288, 11008, 3, 20.9, 22.9),
             (57344, 12288, 4, 77.0, 83.3), (57344, 12288, 12, 82.5, 89.2), (12288, 12288, 3, 25.6, 24.4), (12288, 11008, 16, 28.5, 25.5)]


@pytest.mark.parametrize("m,k,n,six,fewer", SIX_UNITS)
def test_rows_of_six_units_take_the_faster_cut(m, k, n, six, fewer):
    kernel, ranges, *_ = plan("q4", n, m, k, workspace(n, m, k))
    assert kernel == rx.KERNEL_STREAM and (ranges == 1) == (six < fewer)
