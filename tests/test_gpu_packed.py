"""GPU test of the tiled GEMM on packed 4-bit weights where its rounds of 256 columns, its eight scales per round and its tiles end."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def rx():
    from paper_2311_02103_amd import binding
    binding.lib()
    return binding


# a weight is rounded once to fp16, a result once more: below 2 * 2^-11 in the 2-norm
REL = 1e-3


@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("k", [128, 256, 384, 640, 1152])
@pytest.mark.parametrize("m,n", [(4, 65), (68, 130), (260, 193), (1028, 260), (16388, 600)])
def test_ends_of_rounds_and_tiles(rx, m, k, n, group):
    """Rows of half a round and of one and a half, matrices of one granule, scales read up to the last one of the matrix: the codes and
    scales end where their buffers end, and what lies behind them is poison."""
    g = torch.Generator(device="cuda")
    g.manual_seed(m + k + n + group)
    codes = torch.randint(-2 ** 31, 2 ** 31 - 1, (m * k // 8 + 64,), device="cuda", dtype=torch.int32, generator=g)
    scales = torch.full((m * k // group + 64,), float("nan"), device="cuda", dtype=torch.float16)
    scales[:m * k // group] = (torch.rand(m * k // group, device="cuda", generator=g) * 0.01 + 0.001).half()
    q, s = codes[:m * k // 8].view(m, k // 8), scales[:m * k // group].view(m, k // group)
    w = rx.QMat(q, s, m, k, group)
    dense = torch.empty(m, k, dtype=torch.int8, device="cuda")
    rx.check(rx.relax_unpack_int4(w, dense))
    x = torch.randn(n, k, device="cuda", generator=g).half()
    out = torch.full((n + 1, m), float("nan"), device="cuda", dtype=torch.float16)
    assert rx.relax_plan_matmul("q4", n, m, k)[1] == rx.KERNEL_TILED
    rx.check(rx.relax_dequant_matmul(x, w, out, n))
    want = x.double() @ (dense.double() * s.double().repeat_interleave(group, 1)).t()
    assert float((out[:n].double() - want).norm() / want.norm()) < REL
    assert bool(out[n].isnan().all())
