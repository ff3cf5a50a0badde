"""GPU tests of relax_attention: calls that carry decode rows beside a prompt chunk (the prefill kernel's form for sequences with one row), and
calls of decode rows alone with grouped heads."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# A wavefront step is 16 tokens (heads of 128, eight wavefronts: 128 a round; heads of 64 the same): lengths around steps and rounds, wavefronts with no
# token, one step, an odd and an even number of steps.
LENGTHS = [1, 2, 15, 16, 17, 127, 128, 129, 255, 256, 257, 300, 384, 511, 640, 1000]


@pytest.mark.parametrize("h,g,d", [(4, 4, 128), (8, 2, 128), (6, 2, 64), (4, 4, 64)])
@pytest.mark.parametrize("first", [True, False])
def test_decode_rows_beside_a_prompt_against_float64(h, g, d, first):
    prompt = (40, 200)
    _check(h, g, d, [prompt] + [(1, L) for L in LENGTHS] if first else [(1, L) for L in LENGTHS[::-1]] + [prompt, (1, 3)])


# Tiles of 32 tokens, four wavefronts, splits of up to 512 tokens: lengths around each; the largest group of query heads, and heads of 64
@pytest.mark.parametrize("h,g,d", [(16, 2, 128), (16, 1, 128), (16, 4, 64)])
def test_grouped_decode_rows_against_float64(h, g, d):
    _check(h, g, d, [(1, L) for L in (1, 31, 32, 33, 64, 65, 96, 127, 128, 129, 160, 511, 512, 513, 1000)])


# 64 queries and four KV groups per workgroup (few workgroups, more than 64 rows or 400 tokens) and the calls next to them
@pytest.mark.parametrize("h,g,d", [(4, 4, 128), (8, 2, 128), (4, 2, 64)])
@pytest.mark.parametrize("seqs", [[(65, 65)], [(64, 399)], [(64, 400)], [(64, 448)], [(64, 449)], [(17, 1000)], [(16, 463)], [(100, 129)], [(128, 1000)], [(129, 257)], [(512, 1000)],
                                  [(70, 70), (2, 600), (1, 1), (1, 500)]])
def test_few_tiles_against_float64(h, g, d, seqs):
    _check(h, g, d, seqs)


def _check(h, g, d, seqs):
    from paper_2311_02103_amd import binding as rx
    cap = 1024
    q_lens, kv_lens = [s[0] for s in seqs], [s[1] for s in seqs]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * d + g)
    B, n = len(seqs), sum(q_lens)
    q, k, v = (torch.randn(shape, device="cuda", generator=gen).half() for shape in ((n, h, d), (B, cap, g, d), (B, cap, g, d)))
    for b, L in enumerate(kv_lens):                       # what lies behind a sequence must not be read into it
        k[b, L:], v[b, L:] = float("nan"), float("inf")
    q[-1] *= 30.0                                         # one row with large scores
    dims = rx.make_dims(h * d, h, g, d, 64, cap, B)
    rope = torch.empty(rx.relax_rope_table_bytes(dims) // 4, dtype=torch.float32, device="cuda")
    rx.check(rx.relax_rope_table_init(dims, rope))
    ws_bytes = rx.relax_workspace_bytes(dims, n, max(kv_lens), B)
    ws, out = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"), torch.full_like(q, float("nan"))
    rx.check(rx.relax_attention(q, rx.KVCache(k, v, rope), rx.Seqs(q_lens, kv_lens), dims, out, n, ws, ws_bytes))
    row = 0
    for b, (ql, L) in enumerate(seqs):
        kk, vv = (t[b, :L].double().repeat_interleave(h // g, 1).transpose(0, 1).contiguous() for t in (k, v))
        s = q[row:row + ql].double().transpose(0, 1).contiguous() @ kk.transpose(1, 2).contiguous() / math.sqrt(d)
        s = s.masked_fill(torch.arange(L, device="cuda")[None] > torch.arange(L - ql, L, device="cuda")[:, None], -math.inf)
        want = (torch.softmax(s, 2) @ vv).transpose(0, 1)
        got = out[row:row + ql].double()
        # one rounding to fp16 (2^-11), for the prompt's rows one of the weights too
        assert float((got - want).norm() / want.norm()) < 1e-3, (b, ql, L)
        row += ql
