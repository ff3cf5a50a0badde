"""GPU tests of the few-row matmuls, above all the streaming kernel (fewrow_kernel.h), at the sizes where its tiling can go wrong:
rows of x around the blocks of 16, weight rows that do not fill a row tile, columns that do not divide over the wavefronts, one k
range in all weight formats, several with more row tiles than LDS holds; and of the layers that run on it."""
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


def _packed(rx, fmt, m, k, group, g):
    """(QMat, its values in float64): random codes, scales 0.001 .. 0.011."""
    words = k // 8 if fmt == "q4" else 3 * k // 32
    q = torch.randint(-2 ** 31, 2 ** 31 - 1, (m, words), device="cuda", dtype=torch.int32, generator=g)
    s = (torch.rand(m, k // group, device="cuda", generator=g) * 0.01 + 0.001).half()
    w = rx.QMat(q, s, m, k, group)
    codes = torch.empty(m, k, dtype=torch.int8, device="cuda")
    rx.check((rx.relax_unpack_int4 if fmt == "q4" else rx.relax_unpack_q3_native)(w, codes))
    return w, codes.double() * s.double().repeat_interleave(group, 1)


# m: below, at and beside a row tile of 16, one that needs several tiles per workgroup; k: one unit, units that leave wavefronts
# idle or uneven, the 7B / 13B / 70B rows.  Which kernel a row count takes is the dispatch's choice here (3-bit calls have one k
# range; 30000 and 4100 rows of 4-bit weights go to the split-K kernel); the tests below say which one they reach.
SHAPES = [(4, 256), (20, 512), (520, 4096), (72, 11008), (36, 13824), (40, 28672), (30000, 1024), (4100, 8192)]
# A weight is rounded once to fp16 (2^-11 of its value, the final multiply of the decode), a result once more; sums of k terms with
# random signs keep the relative 2-norm error at that of one term: below 2 * 2^-11 = 1e-3.
REL = 1e-3


@pytest.mark.parametrize("m,k", SHAPES)
@pytest.mark.parametrize("fmt,group", [("q4", 32), ("q4", 64), ("q4", 128), ("q3", 32)])
def test_packed_formats_against_float64(rx, fmt, group, m, k):
    if fmt == "q3" and k > 12288:
        pytest.skip("the 3-bit call takes rows of at most 12288 columns at these row counts")
    g = _gen(m + k + group)
    w, ref = _packed(rx, fmt, m, k, group, g)
    ws_bytes = rx.relax_matmul_workspace_bytes(w, 128) if fmt == "q4" else 0
    ws = torch.empty(max(16, ws_bytes), dtype=torch.uint8, device="cuda")
    for n in (2, 15, 16, 17, 32, 33, 64):
        x = torch.randn(n, k, device="cuda", generator=g).half()
        out = torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
        if fmt == "q4":
            rx.check(rx.relax_dequant_matmul(x, w, out, n, ws, ws_bytes))
        else:
            rx.check(rx.relax_dequant_matmul_q3_native(x, w, out, n))
        want = x.double() @ ref.t()
        assert torch.isfinite(out.float()).all()
        assert float((out.double() - want).norm() / want.norm()) < REL, (fmt, group, m, k, n)


@pytest.mark.parametrize("m,k", [(4, 128), (20, 384), (520, 4096), (72, 8192), (3000, 5120)])
def test_half_weights_against_float64(rx, m, k):
    g = _gen(m + k)
    w = torch.randn(m, k, device="cuda", generator=g).half() * 0.05
    for n in (2, 15, 16, 17, 32):
        x = torch.randn(n, k, device="cuda", generator=g).half()
        out = torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
        rx.check(rx.relax_half_matmul(x, w, out, n, m, k))
        want = x.double() @ w.double().t()
        assert float((out.double() - want).norm() / want.norm()) < REL, (m, k, n)


def test_infinities_stay_in_their_row(rx):
    """A row of x with an infinity and a weight row with one change their own results only (dead units, lanes past the end of a
    row and rows past n contribute nothing, not 0 * inf)."""
    m, k, n = 40, 384, 5
    g = _gen(3)
    w = torch.randn(m, k, device="cuda", generator=g).half() * 0.05
    x = torch.randn(n, k, device="cuda", generator=g).half()
    clean = torch.empty(n, m, device="cuda", dtype=torch.float16)
    rx.check(rx.relax_half_matmul(x, w, clean, n, m, k))
    w[7, 5], x[2, 300] = float("inf"), float("inf")
    out = torch.empty_like(clean)
    rx.check(rx.relax_half_matmul(x, w, out, n, m, k))
    rows, cols = torch.arange(n) != 2, torch.arange(m) != 7
    assert torch.equal(out[rows][:, cols], clean[rows][:, cols])
    assert not torch.isfinite(out[2].float()).any() and not torch.isfinite(out[:, 7].float()).any()


LAYERS = [wl.LayerShape("mha-64", hidden=512, n_heads=8, n_kv_heads=8, head_dim=64, ffn=1024),
          wl.LayerShape("gqa-128", hidden=1024, n_heads=8, n_kv_heads=2, head_dim=128, ffn=2816)]


@pytest.mark.parametrize("si", range(len(LAYERS)))
@pytest.mark.parametrize("fmt", ["q4", "q3", "f16"])
def test_layers_on_it_against_the_first_rows_of_a_larger_call(rx, fmt, si):
    """Rotary + append, residuals and SwiGLU as its epilogues (2 .. 64 rows) against the launches of their own of a call with
    more rows than it takes: prefixes of one prompt, whose rows depend on earlier rows only."""
    from paper_2311_02103_amd.runtime import DeviceLayer, DeviceLayerF16, DeviceLayerQ3
    shape, n_all = LAYERS[si], 200
    sizes = dict(hidden=shape.hidden, n_heads=shape.n_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim, ffn=shape.ffn, kv_capacity=256, n_max=n_all)
    if fmt == "q4":
        layer = DeviceLayer(wl.layer_weights(shape, 4), **sizes)
    elif fmt == "q3":
        layer = DeviceLayerQ3(wl.layer_weights3(shape, 4), **sizes)
    else:
        host = {name: wl.normal_f16_bits(4, i, mk, std=0.02) for i, (name, mk) in enumerate(shape.matrices().items())}
        host.update({name: wl.normal_f16_bits(4, 10 + i, (shape.hidden,), std=0.1, mean=1.0) for i, name in enumerate(("norm_attn", "norm_ffn"))})
        layer = DeviceLayerF16(host, **sizes)
    x = torch.from_numpy(wl.activations(shape, 4, 0, n_all).view(np.int16)).view(torch.float16).cuda()
    want, k_all, v_all = layer.forward(x, [n_all], [n_all]).double(), layer.k.clone(), layer.v.clone()
    for n in (2, 5, 16, 17, 40, 64):
        layer.k.zero_(), layer.v.zero_()
        got = layer.forward(x[:n].contiguous(), [n], [n]).double()
        # seven fp16 roundings (2^-11 each) on each side, independent where the two paths round at other points
        assert float((got - want[:n]).norm() / want[:n].norm()) < 4e-3, (fmt, n)
        for a, b in ((layer.k, k_all), (layer.v, v_all)):
            assert float((a[0, :n].double() - b[0, :n].double()).norm() / b[0, :n].double().norm()) < 2e-3
            assert not a[0, n:].any()


def _shifted(t, elements):
    """A copy of t that starts `elements` elements into its storage."""
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device="cuda")
    buf[elements:] = t.reshape(-1)
    return buf[elements:].view(t.shape)


@pytest.mark.parametrize("shift_q,shift_s", [(1, 0), (0, 2), (2, 4)])
def test_unaligned_4bit_weights_keep_their_fp32_scales(rx, shift_q, shift_s):
    """Codes or scales that are aligned to 4 or 8 bytes only (views into one packed checkpoint) are served by the matvec kernels at 2
    to 15 rows, with or without a workspace: the same bits, scales applied in fp32."""
    m, k, g = 512, 1024, _gen(9)
    w, _ = _packed(rx, "q4", m, k, 32, g)
    w = rx.QMat(_shifted(w.q, shift_q), _shifted(w.s, shift_s), m, k, 32)
    ws_bytes = rx.relax_matmul_workspace_bytes(w, 64)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    for n in (2, 5, 15):
        x = torch.randn(n, k, device="cuda", generator=g).half()
        with_ws, without = torch.empty(n, m, device="cuda", dtype=torch.float16), torch.empty(n, m, device="cuda", dtype=torch.float16)
        rx.check(rx.relax_dequant_matmul(x, w, with_ws, n, ws, ws_bytes))
        rx.check(rx.relax_dequant_matmul(x, w, without, n, None, 0))
        assert torch.equal(with_ws, without), n


def test_layer_on_unaligned_4bit_weights_runs_on_the_matvec_kernels(rx):
    from paper_2311_02103_amd.runtime import DeviceLayer
    shape = LAYERS[0]
    layer = DeviceLayer(wl.layer_weights(shape, 4), hidden=shape.hidden, n_heads=shape.n_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim,
                        ffn=shape.ffn, kv_capacity=64, n_max=16)
    for mat in (layer.weights.wqkv, layer.weights.wo, layer.weights.wgu, layer.weights.wdown):
        mat.q, mat.s = _shifted(mat.q, 1), _shifted(mat.s, 2)
    x = torch.from_numpy(wl.activations(shape, 4, 0, 15).view(np.int16)).view(torch.float16).cuda()
    for n in (5, 15):
        got = layer.forward(x[:n].contiguous(), [n], [n])
        try:                                              # the switch that keeps every call on the matvec kernels
            rx.check(rx.relax_set_option("layer_matvec_rows", 64))
            want = layer.forward(x[:n].contiguous(), [n], [n])
        finally:
            rx.check(rx.relax_set_option("layer_matvec_rows", 4))
        assert torch.equal(got, want), n


@pytest.mark.parametrize("low,high", [(2.0 ** -24, 2.0 ** -14), (2.0 ** -14, 1.0), (1.0, 65504.0), (16384.0, 65504.0)])
def test_3bit_scales_over_the_whole_fp16_range(rx, low, high):
    """2 to 16 rows of 3-bit weights, scales from the smallest subnormal to the largest fp16 value: products are exact, so what is
    left is the fp32 sum (k roundings at most) and the rounding of the result."""
    m, k, g = 64, 512, _gen(11)
    q = torch.randint(-2 ** 31, 2 ** 31 - 1, (m, 3 * k // 32), device="cuda", dtype=torch.int32, generator=g)
    s = torch.exp(torch.empty(m, k // 32, device="cuda").uniform_(float(np.log(low)), float(np.log(high)), generator=g)).clamp(low, high).half()
    w = rx.QMat(q, s, m, k, 32)
    codes = torch.empty(m, k, dtype=torch.int8, device="cuda")
    rx.check(rx.relax_unpack_q3_native(w, codes))
    ref = codes.double() * s.double().repeat_interleave(32, 1)
    for n in (2, 3, 15, 16):
        x = (torch.randn(n, k, device="cuda", generator=g) / min(1.0, 30 * high) if high < 1 else torch.randn(n, k, device="cuda", generator=g) / (16 * high)).half()
        out = torch.empty(n, m, device="cuda", dtype=torch.float16)
        rx.check(rx.relax_dequant_matmul_q3_native(x, w, out, n))
        want, terms = x.double() @ ref.t(), x.double().abs() @ ref.abs().t()
        bound = 2.0 ** -11 * want.abs() + 2.0 ** -25 + k * 2.0 ** -24 * terms           # 2^-25: half of the smallest fp16 step
        assert bool(((out.double() - want).abs() <= bound).all()), n


def _units(k, ranges):
    """Units of 256 columns of the wavefront with most of them."""
    return -(-(k // 256) // (8 * ranges))


def _more_tiles_than_lds(n, m, k, ranges, group):
    """Whether a workgroup of the streaming kernel gets more row tiles than its 152 KB of LDS hold sums of, beside the offsets of 4-bit codes where
    scales meet sums (more than 16 rows; with fewer the sums wait there instead)."""
    blocks, tiles, units = (1 if n <= 16 else 2 if n <= 32 else 4), -(-m // 16), _units(k, ranges)
    offsets = 8 * blocks * -(-units // 4) * 3 * 16 * 1024 // group * 2 if group > 32 and blocks == 2 and units < 3 else 0
    return blocks > 1 and -(-tiles // min(tiles, 256 // ranges)) > (152 * 1024 - offsets) // (8 * blocks * 1024)


# (m, k, n, k ranges, sums flushed inside the loop): blocks of 16, 32 and 64 rows
RANGES = [(20, 5120, 15, 3, False), (20, 28672, 16, 14, False), (20, 6656, 17, 4, False), (11264, 6656, 17, 4, True), (11264, 8192, 32, 4, True),
          (12292, 11008, 17, 3, True), (20, 5120, 33, 3, False), (11264, 4096, 33, 2, True), (16388, 2816, 64, 2, True), (11264, 5632, 48, 3, True)]


# Groups of 64 and 128 up to 32 rows: one and two units of 32 x rows with scales on sums, three with scales on codes
RANGES_COARSE = [(20, 5120, 15, 3, False), (20, 28672, 16, 8, False), (20, 6656, 17, 4, False), (11264, 6656, 17, 2, False), (12292, 11008, 32, 3, True),
                 (16400, 8192, 17, 2, True), (16400, 8192, 32, 2, True), (20500, 11008, 17, 2, True)]


@pytest.mark.parametrize("group,m,k,n,ranges,flush", [(32,) + r for r in RANGES] +
                         [(g,) + r for g in (64, 128) for r in RANGES_COARSE + [r for r in RANGES if r[2] > 32]])
def test_several_k_ranges_against_float64(rx, group, m, k, n, ranges, flush):
    g = _gen(m + k + n)
    w, ref = _packed(rx, "q4", m, k, group, g)
    size = rx.relax_matmul_workspace_bytes(w, 128)
    assert rx.relax_plan_matmul("q4", n, m, k, size, group)[:3] == (rx.OK, rx.KERNEL_STREAM, ranges) and _more_tiles_than_lds(n, m, k, ranges, group) == flush
    ws = torch.full((size + 4096,), 7, dtype=torch.uint8, device="cuda")
    x = torch.randn(n, k, device="cuda", generator=g).half()
    out = [torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16) for _ in range(2)]
    for o in out:
        rx.check(rx.relax_dequant_matmul(x, w, o, n, ws, size))
    want = x.double() @ ref.t()
    assert float((out[0].double() - want).norm() / want.norm()) < REL
    assert torch.equal(out[0], out[1]) and bool((ws[size:] == 7).all())


@pytest.mark.parametrize("fmt,m,k,n", [("q3", 520, 4096, 15), ("q3", 72, 11008, 2), ("q3", 3000, 5120, 17), ("q3", 520, 2048, 64),
                                       ("f16", 520, 4096, 16), ("f16", 3000, 4096, 32), ("f16", 72, 8192, 3), ("f16", 4100, 12288, 2)])
def test_one_k_range_of_the_other_formats(rx, fmt, m, k, n):
    """... reaches the streaming kernel (fp16 rows of 12288 columns have no instance of it); 3-bit codes and scales aligned to 4 bytes."""
    g = _gen(m + k + n)
    x = torch.randn(n, k, device="cuda", generator=g).half()
    out = torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
    assert rx.relax_plan_matmul(fmt, n, m, k)[:2] == (rx.OK, rx.KERNEL_MATVEC if k == 12288 else rx.KERNEL_STREAM)
    if fmt == "q3":
        w, ref = _packed(rx, fmt, m, k, 32, g)
        w = rx.QMat(_shifted(w.q, 1), _shifted(w.s, 2), m, k, 32)
        rx.check(rx.relax_dequant_matmul_q3_native(x, w, out, n))
    else:
        w = torch.randn(m, k, device="cuda", generator=g).half() * 0.05
        ref = w.double()
        rx.check(rx.relax_half_matmul(x, w, out, n, m, k))
    want = x.double() @ ref.t()
    assert float((out.double() - want).norm() / want.norm()) < REL


def test_fp16_instances_leave_out_seven_units_per_wavefront(rx):
    """One k range of 6145 to 7168 columns would need it: these rows take the kernels they took without the streaming kernel."""
    for k, stream in ((6144, True), (6656, False), (7168, False), (7296, True), (8192, True)):
        assert (rx.relax_plan_matmul("f16", 16, 4096, k)[1] == rx.KERNEL_STREAM) == stream, k


@pytest.mark.parametrize("fmt,shape,rows", [("q3", wl.LLAMA7B, (17, 33, 64)), ("f16", wl.LLAMA7B, (17, 32)),
                                            ("q4", wl.LayerShape("w13b", hidden=5120, n_heads=40, n_kv_heads=40, head_dim=128, ffn=13824), (17, 32, 64))])
def test_wide_layers_against_the_first_rows_of_a_larger_call(rx, fmt, shape, rows):
    """Partial rows in workspace that is dead at that point, and more row tiles than LDS holds: the down projection in fp16 and the QKV
    and gate/up projections of 33 rows and more in 3 bits run several k ranges.  As above, on random codes."""
    from paper_2311_02103_amd.runtime import DeviceLayer, DeviceLayerF16, DeviceLayerQ3
    n_all, r, host = 130, np.random.RandomState(7), {}
    for name, (m, k) in shape.matrices().items():
        if fmt == "f16":
            host[name] = (r.standard_normal((m, k)).astype(np.float32) * 0.02).astype(np.float16).view(np.uint16)
        else:
            host[name + ".q"] = r.randint(0, 2 ** 32, (m, k // 8 if fmt == "q4" else 3 * k // 32), dtype=np.uint32)
            host[name + ".s"] = (r.random_sample((m, k // 32)) * 0.006 + 0.001).astype(np.float16).view(np.uint16)
    host.update({name: wl.normal_f16_bits(4, 10 + i, (shape.hidden,), std=0.1, mean=1.0) for i, name in enumerate(("norm_attn", "norm_ffn"))})
    layer = {"q4": DeviceLayer, "q3": DeviceLayerQ3, "f16": DeviceLayerF16}[fmt](
        host, hidden=shape.hidden, n_heads=shape.n_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim, ffn=shape.ffn, kv_capacity=192, n_max=n_all)
    x = torch.from_numpy(wl.activations(shape, 4, 0, n_all).view(np.int16)).view(torch.float16).cuda()
    want, k_all = layer.forward(x, [n_all], [n_all]).double(), layer.k.clone()
    for n in rows:
        layer.k.zero_(), layer.v.zero_()
        got = layer.forward(x[:n].contiguous(), [n], [n]).double()
        assert float((got - want[:n]).norm() / want[:n].norm()) < 4e-3, (fmt, n)
        assert float((layer.k[0, :n].double() - k_all[0, :n].double()).norm() / k_all[0, :n].double().norm()) < 2e-3


# Rows around a tile, whole and ragged slices; units per wavefront at 2 (1: some wavefronts without any), 5 and 16 rows, and at 17 and 32 of groups of
# 64 and 128 (three units of 32 rows of x take their scales on codes); 0: the groups differ
EXACT_Q4 = [(20, 256, (1, 1, 1), (1, 1)), (40, 1280, (1, 1, 1), (1, 1)), (72, 4352, (3, 3, 1), (1, 1)), (520, 8192, (1, 1, 1), (1, 1)), (36, 9984, (5, 1, 1), (1, 1)),
            (40, 13824, (2, 1, 1), (1, 1)), (8200, 4096, (2, 2, 2), (2, 2)), (12292, 6144, (3, 3, 0), (3, 3)), (12292, 6656, (4, 4, 0), (2, 2)),
            (12292, 9984, (5, 5, 1), (3, 2)), (40976, 8192, (4, 4, 4), (2, 2))]


@pytest.mark.parametrize("m,k,units,units_32", EXACT_Q4)
@pytest.mark.parametrize("group", [32, 64, 128])
def test_4bit_scales_meet_fp32_sums(rx, group, m, k, units, units_32):
    """Up to 16 rows of groups of 32 and 32 rows of longer ones are exact but for the fp32 sums and the rounding of the result, for scales of any size,
    for x far from zero and for small x: the codes go in as u + 64, so a group's terms are at most 79 / 8 of those of its largest codes."""
    g = _gen(m + k + group)
    w, _ = _packed(rx, "q4", m, k, group, g)
    codes = torch.empty(m, k, dtype=torch.int8, device="cuda")
    rx.check(rx.relax_unpack_int4(w, codes))
    size = rx.relax_matmul_workspace_bytes(w, 64)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    for low, high, mean, std in ((2.0 ** -24, 2.0 ** -14, 0.0, 1.0), (2.0 ** -8, 1.0, 0.5, 0.01), (1e-3, 1e-2, 0.0, 3e-4)):
        s = torch.exp(torch.empty(m, k // group, device="cuda").uniform_(float(np.log(low)), float(np.log(high)), generator=g)).clamp(low, high).half()
        w = rx.QMat(w.q, s, m, k, group)
        ref = codes.double() * s.double().repeat_interleave(group, 1)
        largest = 79 * s.double().repeat_interleave(group, 1)
        for n, want_units in list(zip((2, 5, 16), units)) + (list(zip((17, 32), units_32)) if group > 32 else []):
            _, kernel, ranges, *_ = rx.relax_plan_matmul("q4", n, m, k, size, group)
            if kernel != rx.KERNEL_STREAM and want_units == 0:                        # (the split-K kernel takes it)
                continue
            assert kernel == rx.KERNEL_STREAM and (want_units == 0 or _units(k, ranges) == want_units)
            if n > 16 and want_units > 2:
                continue
            x = (torch.randn(n, k, device="cuda", generator=g) * std + mean).half()
            out = torch.empty(n, m, device="cuda", dtype=torch.float16)
            rx.check(rx.relax_dequant_matmul(x, w, out, n, ws, size))
            want, terms = x.double() @ ref.t(), x.double().abs() @ largest.t()
            # 2^-25: half of the smallest fp16 step; at most 128 roundings lie on the way of a term (MFMAs of its group, its wavefront's groups, wavefronts)
            bound = 2.0 ** -11 * want.abs() + 2.0 ** -25 + 128 * 2.0 ** -24 * terms
            assert bool(((out.double() - want).abs() <= bound).all()), (n, low)


@pytest.mark.parametrize("group", [32, 64, 128])
def test_4bit_infinite_scales_stay_in_their_row(rx, group):
    """... also next to units that a wavefront does not have, where the scales of the next row lie."""
    m, k, n, g = 40, 1280, 5, _gen(5)
    w, _ = _packed(rx, "q4", m, k, group, g)
    size = rx.relax_matmul_workspace_bytes(w, 64)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    x = torch.randn(n, k, device="cuda", generator=g).half()
    clean, out = (torch.empty(n, m, device="cuda", dtype=torch.float16) for _ in range(2))
    rx.check(rx.relax_dequant_matmul(x, w, clean, n, ws, size))
    s = w.s.clone()
    s[7, 0], s[20] = float("inf"), float("nan")
    rx.check(rx.relax_dequant_matmul(x, rx.QMat(w.q, s, m, k, group), out, n, ws, size))
    rows = (torch.arange(m) != 7) & (torch.arange(m) != 20)
    assert torch.equal(out[:, rows], clean[:, rows])
    assert not torch.isfinite(out[:, ~rows].float()).any()


# (the last one takes its sums out of LDS inside the loop where groups are long)
@pytest.mark.parametrize("m,k", [(40, 1280), (24, 13824), (16400, 8192)])
@pytest.mark.parametrize("n", [5, 16, 32])
@pytest.mark.parametrize("group", [32, 64, 128])
def test_4bit_infinite_x_keeps_its_sign(rx, group, n, m, k):
    """An infinity in x times a code is an infinity of that sign, times code 0 a NaN, however the codes' offset is taken out; and the row's alone."""
    g = _gen(m + k + group)
    w, ref = _packed(rx, "q4", m, k, group, g)
    size = rx.relax_matmul_workspace_bytes(w, 64)
    assert rx.relax_plan_matmul("q4", n, m, k, size, group)[1] == rx.KERNEL_STREAM
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    x = torch.randn(n, k, device="cuda", generator=g).half()
    clean, out = (torch.empty(n, m, device="cuda", dtype=torch.float16) for _ in range(2))
    rx.check(rx.relax_dequant_matmul(x, w, clean, n, ws, size))
    inf = float("inf")
    x[1, 77], x[2, k - 1], x[n - 1, 300], x[3, 5] = inf, -inf, inf, float("nan")
    rx.check(rx.relax_dequant_matmul(x, w, out, n, ws, size))
    for i, column, sign in ((1, 77, 1.0), (2, k - 1, -1.0), (n - 1, 300, 1.0)):
        want = (ref[:, column] * (sign * inf)).half()
        assert torch.equal(torch.isnan(out[i]), torch.isnan(want)), i
        assert torch.equal(out[i][~torch.isnan(want)], want[~torch.isnan(want)]), i
    assert torch.isnan(out[3]).all()
    others = [i for i in range(n) if i not in (1, 2, 3, n - 1)]
    assert torch.equal(out[others], clean[others])


# Weights of the last one: a layer whose three and four rows the streaming kernel takes from the matvec kernels
FUSED = [(LAYERS[0], 32, 0), (LAYERS[1], 32, 0), (LAYERS[1], 128, 0), (wl.LayerShape("w", hidden=5120, n_heads=40, n_kv_heads=8, head_dim=128, ffn=13824), 128, 96)]


@pytest.mark.parametrize("shape,group,matvec_mb", FUSED)
def test_fused_light_steps_change_no_bit_at_two_to_four_rows(rx, shape, group, matvec_mb):
    """fuse_finish on and off, on the matrix path (matvec_mb = 0: in place of the matvec kernels) and for the calls that it takes by itself."""
    from paper_2311_02103_amd.runtime import DeviceLayer
    layer = DeviceLayer(_random_layer(shape, group), hidden=shape.hidden, n_heads=shape.n_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim,
                        ffn=shape.ffn, kv_capacity=64, n_max=16, group=group)
    x = torch.from_numpy(wl.activations(shape, 4, 0, 4).view(np.int16)).view(torch.float16).cuda()
    try:
        rx.check(rx.relax_set_option("layer_matvec_mb", matvec_mb))
        for n in (2, 3, 4):
            rx.check(rx.relax_set_option("layer_matvec_rows", 1 if n == 2 and matvec_mb == 0 else 4))
            got = []
            for fused in (0, 1):
                rx.check(rx.relax_set_option("fuse_finish", fused))
                layer.k.zero_(), layer.v.zero_()
                got.append((layer.forward(x[:n].contiguous(), [n], [n]).clone(), layer.k.clone(), layer.v.clone()))
            for a, b in zip(*got):
                assert torch.equal(a.view(torch.int16), b.view(torch.int16)), n
    finally:
        for name, value in (("layer_matvec_mb", 96), ("layer_matvec_rows", 4), ("fuse_finish", 1)):
            rx.check(rx.relax_set_option(name, value))


@pytest.mark.parametrize("shape,group,rows_switch,matvec", [(LAYERS[0], 32, 4, True), (LAYERS[1], 128, 4, True), (FUSED[3][0], 128, 4, False),
                                                            (FUSED[3][0], 128, 64, True)])
def test_three_and_four_rows_leave_the_matvec_kernels_in_large_layers_only(rx, shape, group, rows_switch, matvec):
    """A rotary table aligned to 8 bytes keeps a call on the matvec kernels: the same bits where an aligned one stays there too, close to them where not."""
    from paper_2311_02103_amd.runtime import DeviceLayer
    layer = DeviceLayer(_random_layer(shape, group), hidden=shape.hidden, n_heads=shape.n_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim,
                        ffn=shape.ffn, kv_capacity=64, n_max=16, group=group)
    x = torch.from_numpy(wl.activations(shape, 4, 0, 4).view(np.int16)).view(torch.float16).cuda()
    try:
        rx.check(rx.relax_set_option("layer_matvec_rows", rows_switch))
        got = [layer.forward(x[:n].contiguous(), [n], [n]).clone() for n in (3, 4)]
        layer.cache = rx.KVCache(layer.k, layer.v, _shifted(layer.rope, 2))
        want = [layer.forward(x[:n].contiguous(), [n], [n]) for n in (3, 4)]
    finally:
        rx.check(rx.relax_set_option("layer_matvec_rows", 4))
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)) == matvec
        # seven fp16 roundings (2^-11 each) on each side, independent where the two paths round at other points
        assert float((a.double() - b.double()).norm() / b.double().norm()) < 4e-3


def _random_layer(shape, group):
    r, host = np.random.RandomState(7), {}
    for name, (m, k) in shape.matrices().items():
        host[name + ".q"] = np.frombuffer(bytearray(r.bytes(m * k // 2)), dtype=np.uint32).reshape(m, k // 8)
        host[name + ".s"] = (r.random_sample((m, k // group)) * 0.006 + 0.001).astype(np.float16).view(np.uint16)
    host.update({name: wl.normal_f16_bits(4, 10 + i, (shape.hidden,), std=0.1, mean=1.0) for i, name in enumerate(("norm_attn", "norm_ffn"))})
    return host


# Six units per wavefront and fewer (wavefronts with 5 and 6), row tiles that end early
@pytest.mark.parametrize("m,k,n,group", [(20, 11008, 2, 32), (520, 10496, 3, 32), (4096, 11008, 4, 64), (4096, 11008, 4, 128), (12288, 12288, 2, 32)])
def test_six_units_per_wavefront_against_float64(rx, m, k, n, group):
    g = _gen(m + k + n)
    w, ref = _packed(rx, "q4", m, k, group, g)
    size = rx.relax_matmul_workspace_bytes(w, 64)
    assert rx.relax_plan_matmul("q4", n, m, k, size, group)[:3] == (rx.OK, rx.KERNEL_STREAM, 1)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    x = torch.randn(n, k, device="cuda", generator=g).half()
    out = torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16)
    rx.check(rx.relax_dequant_matmul(x, w, out, n, ws, size))
    want = x.double() @ ref.t()
    assert float((out.double() - want).norm() / want.norm()) < REL


# 17 to 19 row tiles per workgroup, or 34 to 38 of one cut in two: more than the LDS holds shares of beside the offsets, sums wait there inside the loop.  One
# to four units per wavefront; the last row tile has 4 rows.
@pytest.mark.parametrize("m,k,ranges", [(77748, 1536, 1), (73732, 4096, 1), (77748, 4352, 1), (69652, 6400, 1), (73732, 8192, 1), (38836, 14336, 2)])
@pytest.mark.parametrize("group", [32, 64, 128])
def test_more_row_tiles_than_lds_in_one_block_of_rows(rx, group, m, k, ranges):
    n, g = 5, _gen(m + k)
    w, ref = _packed(rx, "q4", m, k, group, g)
    size = rx.relax_matmul_workspace_bytes(w, 16)
    assert rx.relax_plan_matmul("q4", n, m, k, size, group)[:3] == (rx.OK, rx.KERNEL_STREAM, ranges)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    x = torch.randn(n, k, device="cuda", generator=g).half()
    out = [torch.full((n, m), float("nan"), device="cuda", dtype=torch.float16) for _ in range(3)]
    for o in out[:2]:
        rx.check(rx.relax_dequant_matmul(x, w, o, n, ws, size))
    want = x.double() @ ref.t()
    # exact but for the rounding of the result (2^-11 of it at most, 0.4 of that in the norm) and fp32 sums
    assert float((out[0].double() - want).norm() / want.norm()) < 2.5e-4 and torch.equal(out[0], out[1])
    x[1, 7] = float("inf")
    rx.check(rx.relax_dequant_matmul(x, w, out[2], n, ws, size))
    infinite = (ref[:, 7] * float("inf")).half()
    assert torch.equal(torch.nan_to_num(out[2][1], nan=0.5), torch.nan_to_num(infinite, nan=0.5))
    assert torch.equal(out[2][[0, 2, 3, 4]], out[0][[0, 2, 3, 4]])
