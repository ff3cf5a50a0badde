"""GPU tests of the tiled GEMM: every tile, k cut and the two-launch form on its own, row counts around the tiles' edges; and of the
attention kernel's token tiles and softmax."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import workloads as wl  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    from paper_2311_02103_amd import binding
    binding.lib()
    return binding


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


# a weight is rounded once to fp16, a result once more: below 2 * 2^-11 in the 2-norm
REL = 1e-3


@pytest.mark.parametrize("m,k,group", [(4096, 4096, 32), (520, 2816, 64), (1000, 1024, 128), (8192, 2048, 32)])
@pytest.mark.parametrize("with_ws", [True, False])
def test_row_counts_around_the_tile_edges(rx, m, k, group, with_ws):
    g = _gen(m + k)
    q = torch.randint(-2 ** 31, 2 ** 31 - 1, (m, k // 8), device="cuda", dtype=torch.int32, generator=g)
    s = (torch.rand(m, k // group, device="cuda", generator=g) * 0.01 + 0.001).half()
    w = rx.QMat(q, s, m, k, group)
    codes = torch.empty(m, k, dtype=torch.int8, device="cuda")
    rx.check(rx.relax_unpack_int4(w, codes))
    ref = codes.double() * s.double().repeat_interleave(group, 1)
    size = rx.relax_matmul_workspace_bytes(w, 600) if with_ws else 0
    # the workspace ends where it says: nothing behind it may change
    ws = torch.full((size + 4096,), 7, dtype=torch.uint8, device="cuda")
    for n in (65, 129, 192, 193, 256, 257, 300, 384, 385, 511, 512, 513):
        x = torch.randn(n, k, device="cuda", generator=g).half()
        out = torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
        rx.check(rx.relax_dequant_matmul(x, w, out, n, ws if with_ws else None, size))
        want = x.double() @ ref.t()
        assert float((out.double() - want).norm() / want.norm()) < REL, (m, k, n)
        assert bool((ws[size:] == 7).all())


# (m, k, n, tile rows, tile columns, k splits, weight rows of a launch of wide tiles in front); a weight row, and where it can be a row of x,
# beside the edge of a tile
ONE_PASS = [(132, 256, 33, 128, 64, 1, 0), (16388, 256, 65, 128, 128, 1, 0), (16388, 256, 129, 128, 192, 1, 0), (16388, 256, 200, 128, 256, 1, 0),
            (22020, 256, 257, 256, 192, 1, 0), (16388, 256, 600, 256, 256, 1, 0), (16388, 4096, 1200, 128, 256, 1, 13056)]
SPLIT = [(132, 1024, 65, 128, 64, 2, 0), (132, 4096, 65, 128, 64, 8, 0), (4100, 2048, 65, 128, 128, 4, 0), (4100, 5632, 128, 128, 128, 5, 0),
         (8196, 4096, 129, 128, 192, 2, 0), (4100, 11008, 129, 128, 192, 6, 0), (8196, 11008, 200, 128, 256, 3, 0), (12292, 11008, 257, 256, 192, 2, 0),
         (16388, 4096, 65, 256, 128, 2, 0)]


@pytest.mark.parametrize("fmt,case", [("q4", c) for c in ONE_PASS + SPLIT] + [("q3", c) for c in ONE_PASS[:6]] + [("f16", c) for c in ONE_PASS[:4]])
def test_every_tile_exactly(rx, fmt, case):
    """Small integers: every sum is a whole number below 2048, so the result is exact whatever the order of the sums."""
    m, k, n, *planned = case
    g = _gen(m + k + n)
    if fmt == "f16":
        w = torch.randint(-8, 8, (m, k), device="cuda", generator=g).half()
        ref, size = w.double(), 0
    else:
        q = torch.randint(-2 ** 31, 2 ** 31 - 1, (m, k // 8 if fmt == "q4" else 3 * k // 32), device="cuda", dtype=torch.int32, generator=g)
        s = torch.randint(1, 3, (m, k // 32), device="cuda", generator=g).half()
        w = rx.QMat(q, s, m, k, 32)
        codes = torch.empty(m, k, dtype=torch.int8, device="cuda")
        rx.check((rx.relax_unpack_int4 if fmt == "q4" else rx.relax_unpack_q3_native)(w, codes))
        ref = codes.double() * s.double().repeat_interleave(32, 1)
        size = rx.relax_matmul_workspace_bytes(w, n) if planned[2] > 1 else 0
    rc, kernel, splits, rows, cols, wide = rx.relax_plan_matmul(fmt, n, m, k, size)
    assert (rc, kernel, [rows, cols, splits, wide]) == (rx.OK, rx.KERNEL_TILED, planned)
    x = torch.zeros(n, k, device="cuda")
    x.scatter_(1, torch.randint(0, k, (n, 20), device="cuda", generator=g), torch.randint(-3, 4, (n, 20), device="cuda", generator=g).float())
    x, out = x.half(), torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
    ws = torch.full((size + 4096,), 7, dtype=torch.uint8, device="cuda")
    if fmt == "q4":
        rx.check(rx.relax_dequant_matmul(x, w, out, n, ws if size else None, size))
    elif fmt == "q3":
        rx.check(rx.relax_dequant_matmul_q3_native(x, w, out, n))
    else:
        rx.check(rx.relax_half_matmul(x, w, out, n, m, k))
    want = x.double() @ ref.t()
    assert float(want.abs().max()) <= 2048 and torch.equal(out.double(), want)
    assert bool((ws[size:] == 7).all())


@pytest.mark.parametrize("d,heads,kv_heads", [(128, 8, 2), (64, 8, 8)])
def test_prefill_attention_around_its_token_tiles(rx, d, heads, kv_heads):
    """Rows and cached lengths around sub-tiles of 32, tiles of 64 tokens and 128 queries, against float64; NaN behind every
    sequence's end must not be read into a result."""
    g = _gen(d)
    cap = 512
    dims = rx.make_dims(heads * d, heads, kv_heads, d, 256, cap, 2)
    rope = torch.empty(rx.relax_rope_table_bytes(dims) // 4, dtype=torch.float32, device="cuda")
    rx.check(rx.relax_rope_table_init(dims, rope))
    for q_len, past, other in ((16, 0, 1), (31, 1, 33), (32, 96, 64), (33, 95, 127), (127, 1, 128), (128, 0, 129), (129, 127, 1), (200, 57, 300), (256, 256, 31), (16, 47, 63), (17, 47, 65), (33, 32, 64)):
        L, n = q_len + past, q_len + 1
        k = torch.randn(2, cap, kv_heads, d, device="cuda", generator=g).half()
        v = torch.randn(2, cap, kv_heads, d, device="cuda", generator=g).half()
        k[0, L:], v[0, L:], k[1, other:], v[1, other:] = (float("nan"),) * 4
        q = torch.randn(n, heads, d, device="cuda", generator=g).half()
        out = torch.full_like(q, float("nan"))
        size = rx.relax_workspace_bytes(dims, n, cap, 2)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        rx.check(rx.relax_attention(q, rx.KVCache(k, v, rope), rx.Seqs([q_len, 1], [L, other]), dims, out, n, ws, size))
        want = torch.empty(n, heads, d, dtype=torch.float64, device="cuda")
        for rows, slot, length in ((slice(0, q_len), 0, L), (slice(q_len, n), 1, other)):
            ql = rows.stop - rows.start
            mask = torch.arange(length, device="cuda")[None] > torch.arange(length - ql, length, device="cuda")[:, None]
            for h in range(heads):
                kh, vh = k[slot, :length, h * kv_heads // heads].double(), v[slot, :length, h * kv_heads // heads].double()
                sc = (q[rows, h].double() @ kh.t() / d ** 0.5).masked_fill(mask, float("-inf"))
                want[rows, h] = torch.softmax(sc, 1) @ vh
        # P rounded to fp16 (2^-11 each, independent), the result once more
        assert float((out.double() - want).norm() / want.norm()) < 1e-3, (q_len, past, other)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("size", [3.0, 30.0, 300.0, 3000.0, 30000.0])
def test_prefill_attention_on_large_scores(rx, d, size):
    """Queries and keys of magnitude size / 2 .. size: dot products up to 1e11, all finite in fp32.  Three heads: keys equal to the
    queries (each row sees mostly itself), keys that grow along the sequence (the reference point moves all the time), one key
    repeated (equal scores: the mean of the values so far)."""
    n, heads = 200, 3
    g = _gen(int(size))
    dims = rx.make_dims(heads * d, heads, heads, d, 256, n, 1)
    rope = torch.empty(rx.relax_rope_table_bytes(dims) // 4, dtype=torch.float32, device="cuda")
    rx.check(rx.relax_rope_table_init(dims, rope))
    q = torch.randn(n, heads, d, device="cuda", generator=g)
    q = (q.sign() * (0.5 + 0.5 * torch.rand(q.shape, device="cuda", generator=g)) * size).half()
    k, v = q.clone(), torch.randn(n, heads, d, device="cuda", generator=g).half()
    k[:, 1] = (k[:, 1].float() * torch.linspace(0.1, 1.0, n, device="cuda")[:, None]).half()
    k[:, 2] = k[0, 2]
    out, bytes_ = torch.full_like(q, float("nan")), rx.relax_workspace_bytes(dims, n, n, 1)
    ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
    rx.check(rx.relax_attention(q, rx.KVCache(k.contiguous(), v, rope), rx.Seqs([n], [n]), dims, out, n, ws, bytes_))
    assert torch.isfinite(out).all()
    future = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for h in range(heads):
        scores = q[:, h].double() @ k[:, h].double().t()
        p = torch.softmax((scores / d ** 0.5).masked_fill(future, float("-inf")), 1)
        # what the fp32 sum of a score's products may be off by (d + 1 roundings) may turn the softmax; P and the result are rounded
        # to fp16, 2^-11 each.  A row is checked where the first stays below the second.
        slack = (q[:, h].double().abs() @ k[:, h].double().abs().t()).max(1).values * (d + 1) * 2.0 ** -24 / d ** 0.5
        top2 = (scores / d ** 0.5).masked_fill(future, float("-inf")).topk(2, 1).values
        clear = (slack < 2.0 ** -11) | (top2[:, 0] - top2[:, 1] > 2 * slack + 10.0) | (torch.arange(n, device="cuda") == 0)
        if h == 2:                                        # equal keys have equal sums, whatever their rounding
            clear[:] = True
        want = p @ v[:, h].double()
        assert clear.sum() > n // 4
        assert float((out[clear, h].double() - want[clear]).norm() / want[clear].norm()) < 1e-3, h
