"""Host tests of the dispatch of the plain matmuls (relax_plan_matmul): which kernel, k cut and tile sizes take."""
import pytest

from paper_2311_02103_amd import binding as rx


def plan(fmt, n, m, k, ws_bytes=0):
    rc, *rest = rx.relax_plan_matmul(fmt, n, m, k, ws_bytes)
    assert rc == rx.OK
    return tuple(rest)


def workspace(n, m, k):
    """What relax_matmul_workspace_bytes gives for a 4-bit matrix (any pointers do)."""
    return rx.relax_matmul_workspace_bytes(rx.QMat(256, 256, m, k, 32), n)


def test_errors():
    assert rx.relax_plan_matmul("q5", 1, 64, 64)[0] == rx.ERR_UNSUPPORTED
    for n, m, k in ((0, 64, 64), (1, 0, 64), (1, 64, 0), (1, 64, 40)):
        assert rx.relax_plan_matmul("q4", n, m, k)[0] == rx.ERR_SHAPE


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
