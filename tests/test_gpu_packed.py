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
@pytest.mark.parametrize("m,n", [(4, 65), (132, 20), (68, 130), (260, 193), (1028, 260), (16388, 600), (4092, 2000)])
def test_ends_of_rounds_and_tiles(rx, m, k, n, group):
    """Rows of half a round and of one and a half, matrices of one granule, scales read up to the last one of the matrix: behind the scales lie NaNs, and
    other words behind the codes change nothing."""
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
    _, kernel, _, rows, cols, _ = rx.relax_plan_matmul("q4", n, m, k)
    assert kernel == rx.KERNEL_TILED and (m != 4092 or (rows, cols) == (256, 128)) and (n != 20 or cols == 64)
    rx.check(rx.relax_dequant_matmul(x, w, out, n))
    want = x.double() @ (dense.double() * s.double().repeat_interleave(group, 1)).t()
    assert float((out[:n].double() - want).norm() / want.norm()) < REL
    assert bool(out[n].isnan().all())
    codes[m * k // 8:] ^= -1
    again = torch.empty(n, m, device="cuda", dtype=torch.float16)
    rx.check(rx.relax_dequant_matmul(x, w, again, n))
    assert torch.equal(again, out[:n])


@pytest.mark.parametrize("m,k", [
    (1048976, 8192),                                        # 4 GiB of codes and 400 rows more
    (4793664, 28672),                                       # more than 2^32 scales
])
def test_matrices_beyond_32_bits_of_offset(rx, m, k):
    """Rows of the first tiles, of the last ones and of the tiles where offsets counted in 32 bits wrap (the others hold what the memory held)."""
    n, group = 65, 32
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    q, s = torch.empty(m, k // 8, dtype=torch.int32, device="cuda"), torch.empty(m, k // group, dtype=torch.float16, device="cuda")
    wraps = [m - 2 ** 32 // (k // 2), 2 ** 32 // (k // group)]
    ranges = sorted({(max(0, min(r - 300, m - 600)), max(0, min(r - 300, m - 600)) + 600) for r in [0, m] + [r for r in wraps if 0 < r < m]})
    x = torch.randn(n, k, device="cuda", generator=g).half()
    for a, b in ranges:
        q[a:b] = torch.randint(-2 ** 31, 2 ** 31 - 1, (b - a, k // 8), device="cuda", dtype=torch.int32, generator=g)
        s[a:b] = (torch.rand(b - a, k // group, device="cuda", generator=g) * 0.01 + 0.001).half()
    out = torch.empty(n, m, device="cuda", dtype=torch.float16)
    assert rx.relax_plan_matmul("q4", n, m, k)[1] == rx.KERNEL_TILED
    rx.check(rx.relax_dequant_matmul(x, rx.QMat(q, s, m, k, group), out, n))
    for a, b in ranges:
        dense = torch.empty(b - a, k, dtype=torch.int8, device="cuda")
        rx.check(rx.relax_unpack_int4(rx.QMat(q[a:b], s[a:b], b - a, k, group), dense))
        want = x.double() @ (dense.double() * s[a:b].double().repeat_interleave(group, 1)).t()
        assert float((out[:, a:b].double() - want).norm() / want.norm()) < REL, (a, b)


@pytest.mark.parametrize("hidden,heads,kv_heads,q_lens,past", [
    (1024, 6, 1, [513], [0]),                               # one prompt; the last tile holds one head
    (1024, 12, 4, [530] + [1] * 20, [37] + [5 * b for b in range(20)]),     # grouped heads, more sequences than ride in kernel arguments
    (1024, 6, 3, [200, 1, 320, 7], [0, 90, 64, 11]),
    (4096, 112, 8, [1200], [3]),                            # two launches: whole rounds of 256 x 256 tiles and 128 x 256 tiles for the rest
])
def test_rotary_epilogue_equals_the_separate_launch(rx, hidden, heads, kv_heads, q_lens, past):
    """Rotary + append in the QKV GEMM's epilogue against the GEMM and rope_append_kernel: output and caches bit for bit."""
    import numpy as np
    from paper_2311_02103_amd.runtime import DeviceLayer
    rng = np.random.default_rng(hidden + heads)
    d, ffn, n = 128, 256, sum(q_lens)
    host = {}
    for name, m, k in (("wqkv", (heads + 2 * kv_heads) * d, hidden), ("wo", hidden, heads * d), ("wgu", 2 * ffn, hidden), ("wdown", hidden, ffn)):
        host[name + ".q"] = rng.integers(0, 2 ** 32, (m, k // 8), dtype=np.uint32)
        host[name + ".s"] = (rng.random((m, k // 32)) * 0.003 + 0.001).astype(np.float16).view(np.uint16)
    for name in ("norm_attn", "norm_ffn"):
        host[name] = np.ones(hidden, np.float16).view(np.uint16)
    kv_lens = [q + p for q, p in zip(q_lens, past)]
    layer = DeviceLayer(host, hidden=hidden, n_heads=heads, n_kv_heads=kv_heads, head_dim=d, ffn=ffn, kv_capacity=max(kv_lens), kv_slots=len(q_lens),
                        n_max=n, rms_eps=1e-5, rope_base=10000.0, group=32)
    x = torch.from_numpy(rng.standard_normal((n, hidden)).astype(np.float16)).cuda()
    results = []
    try:
        for fused in (0, 1):
            rx.check(rx.relax_set_option("fuse_finish", fused))
            for cache in (layer.k, layer.v):
                cache.copy_(torch.arange(cache.numel(), device="cuda").remainder(7).view(cache.shape).half())
            out = layer.forward(x, q_lens, kv_lens)
            results.append([t.clone().view(torch.int16) for t in (out, layer.k, layer.v)])
    finally:
        rx.check(rx.relax_set_option("fuse_finish", 1))
    for a, b in zip(*results):
        assert torch.equal(a, b)
