"""GEMM tiles of many rows against those of few, bit for bit.

A row's arithmetic does not depend on how many rows share a launch, so a
prompt prefilled 64 tokens at a time (the tiles that the oracle parity tests
pin) and in chunks of hundreds or thousands of rows (256-row tiles, partial
last tiles, split-K partials added by the GEMM itself or by its consumer) gives
the same logits and the same K/V, and so does the LM head row by row."""
import pytest

from tests.gpu_common import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgd():
    import paper_2607_20791_amd as m
    return m


def _world(t, seed, d, ffn, hq, hk, V, layers=1):
    g = t.Generator(device="cuda").manual_seed(seed)

    def w(*s, std=0.02):
        return (t.randn(*s, generator=g, device="cuda") * std).bfloat16()
    one = t.ones(d, device="cuda")
    top = {"embed": w(V, d, std=1.0), "final_norm": one, "lm_head": w(V, d)}
    shapes = {"wq": (hq * 128, d), "wk": (hk * 128, d), "wv": (hk * 128, d), "wo": (d, hq * 128),
              "w_gate": (ffn, d), "w_up": (ffn, d), "w_down": (d, ffn)}
    return top, [dict({n: w(*s) for n, s in shapes.items()}, attn_norm=one, ffn_norm=one) for _ in range(layers)]


def _prefill(rgd, t, world, dims, tokens, max_rows):
    d, ffn, hq, hk, V = dims
    B, n = tokens.shape
    top, layers = world
    cfg = rgd.ModelConfig(len(layers), d, hq, hk, 128, ffn, V, rgd.DTYPE_BF16, 1e-5, 500000.0, n)
    m = rgd.Model(cfg, top, layers, max_rows)
    z = lambda *s: t.zeros(s, dtype=t.bfloat16, device="cuda")  # noqa: E731
    kv = rgd.KV(m, B, n, 0, 16, z(len(layers), B, hk, n, 128), z(len(layers), B, hk, (n + 63) // 64, 128, 64),
                z(len(layers), 1, hk, 16, 128), z(len(layers), 1, hk, 128, 16))
    last = t.empty(B, V, device="cuda")
    rgd.prefill_kv(m, kv, tokens, 0, last)
    t.cuda.synchronize()
    return last, kv.prefix_k, kv.prefix_v


# (d, ffn, heads, kv heads, vocab), prompts, tokens, max_rows of the wide run.
# SwiGLU runs 256-row tiles in every chunk of more than 128 rows but that of 513 (one
# partial tile past 256 rows; 2 + 1 tiles and more).  The projections do where there are
# enough workgroups or steps: an uneven split (88 steps over 16 at 513 rows, 22 over
# 4 at 1300), the three segments of QKV at 1000.  They add their splits themselves
# in the chunks of 2100 (a 52-row last tile; 22 steps over 4 and 56 over 8; four and
# eight heads per KV head), 2600 and, at d = 4096, 690 rows.  Rows of several
# prompts in one chunk, with prefix splits of one and of three 64-position tiles.
# The attention walks over the prefix splits in the wide runs of 690, 2600 (eight query heads) and, with 32
# query heads, of 2100 (66 row blocks, two launches; splits of two tiles, 17 of them: partials in LDS,
# registers and memory), 1300 (eight heads per KV head), 2560 (16; 40 splits) and 200 rows (few rows
# left for the tail kernel), and in those of 150 and 70, which have one split.  In runs of
# 64 rows at a time it does so in the first 64 positions only.  The chunks of 150 and
# 70 rows: last rows that go through the LM head prompt by prompt's chunk (held back, in two lots for 70
# prompts) and in place.
CASES = [((1024, 2816, 8, 4, 512), 1, 257, 300), ((1024, 5632, 8, 2, 512), 1, 700, 513),
         ((1024, 1408, 8, 2, 512), 1, 600, 600), ((1024, 3584, 8, 2, 512), 1, 2100, 2100),
         ((1024, 1408, 8, 1, 512), 1, 2100, 2100),
         ((4096, 1152, 32, 8, 512), 3, 230, 700), ((1024, 1408, 8, 8, 512), 2, 1300, 2600),
         ((1024, 1408, 8, 2, 512), 1, 1300, 1300), ((1024, 1408, 8, 2, 512), 1, 1000, 1000),
         ((1024, 1408, 32, 8, 512), 1, 2100, 2100), ((1024, 128, 32, 4, 512), 1, 1300, 1300),
         ((1024, 128, 32, 2, 512), 1, 2560, 2560), ((1024, 128, 32, 8, 512), 4, 200, 256),
         ((1024, 128, 8, 2, 512), 5, 30, 150), ((1024, 128, 8, 2, 512), 70, 1, 70)]


@pytest.mark.parametrize("dims,prompts,n,rows", CASES)
def test_prefill_chunk_size_does_not_matter(rgd, dims, prompts, n, rows):
    """Two layers: the second one's K/V show every row's attention and projections, the logits only the last row's."""
    t = torch()
    world = _world(t, n, *dims, layers=2)
    g = t.Generator(device="cuda").manual_seed(n + 1)
    tokens = t.randint(0, dims[4], (prompts, n), generator=g, device="cuda", dtype=t.int32)
    few = _prefill(rgd, t, world, dims, tokens, 64)
    wide = _prefill(rgd, t, world, dims, tokens, rows)
    for a, b in zip(few, wide):
        assert t.isfinite(a.float()).all() and t.equal(a, b)


@pytest.mark.parametrize("R,V", [(129, 1100), (256, 512), (257, 4), (300, 64), (513, 1348)])
def test_lm_head_rows_alone_and_together(rgd, R, V):
    """Vocabularies that end inside a 64-column group and inside a 512-column workgroup; rows past one tile."""
    t = torch()
    dims = (1024, 128, 1, 1, V)
    top, layers = _world(t, R, *dims)
    m = rgd.Model(rgd.ModelConfig(1, 1024, 1, 1, 128, 128, V, rgd.DTYPE_BF16, 1e-5, 500000.0, 64), top, layers, R)
    h = t.randn(R, 1024, generator=t.Generator(device="cuda").manual_seed(R), device="cuda").bfloat16()
    out = t.full((R + 1, V), -7.0, device="cuda")
    rgd.kernel_lm_head(m, h, out[:R])
    rows = t.empty(R, V, device="cuda")
    for r in range(0, R, 50):
        rgd.kernel_lm_head(m, h[r:r + 50].contiguous(), rows[r:r + 50])
    t.cuda.synchronize()
    assert t.equal(out[:R], rows) and bool((out[R] == -7.0).all())


# vocabularies at which the 256-row tiles take these rows (two rounds of 128-row workgroups or more
# against one): they end inside a 64-column group, at its end and inside a
# 512-column workgroup; two steps of 64 k, and 16; rows of one tile, of a partial second
# and of a partial third
@pytest.mark.parametrize("R,V,d", [(129, 66308, 128), (200, 66112, 1024), (256, 131076, 128), (257, 44100, 1024),
                                   (300, 65476, 384), (512, 44032, 128), (513, 33100, 1024)])
def test_lm_head_on_wide_tiles(rgd, R, V, d):
    t = torch()
    top, layers = _world(t, R, d, 128, 1, 1, V)
    m = rgd.Model(rgd.ModelConfig(1, d, 1, 1, 128, 128, V, rgd.DTYPE_BF16, 1e-5, 500000.0, 64), top, layers, R)
    h = t.randn(R, d, generator=t.Generator(device="cuda").manual_seed(R), device="cuda").bfloat16()
    out, rows = t.full((R + 1, V), -7.0, device="cuda"), t.empty(R, V, device="cuda")
    rgd.kernel_lm_head(m, h, out[:R])
    for r in range(0, R, 64):
        rgd.kernel_lm_head(m, h[r:r + 64], rows[r:r + 64])
    t.cuda.synchronize()
    assert t.equal(out[:R], rows) and bool((out[R] == -7.0).all())


@pytest.mark.parametrize("R,d,V", [(300, 1024, 65476), (130, 2048, 66308)])
def test_lm_head_of_hidden_states_at_any_element(rgd, R, d, V):
    """Hidden states at 2-, 8- and 16-byte offsets: the 256-row tiles copy 16-byte pieces of aligned rows only."""
    t = torch()
    top, layers = _world(t, R, d, 128, 1, 1, V)
    m = rgd.Model(rgd.ModelConfig(1, d, 1, 1, 128, 128, V, rgd.DTYPE_BF16, 1e-5, 500000.0, 64), top, layers, R)
    h = t.randn(R, d, generator=t.Generator(device="cuda").manual_seed(R), device="cuda").bfloat16()
    want, got = t.empty(R, V, device="cuda"), t.empty(R, V, device="cuda")
    rgd.kernel_lm_head(m, h, want)
    for off in (1, 4, 8):
        at = t.empty(R * d + 8, dtype=t.bfloat16, device="cuda")[off:off + R * d].view(R, d)
        at.copy_(h)
        rgd.kernel_lm_head(m, at, got.zero_())
        t.cuda.synchronize()
        assert t.equal(got, want), off


@pytest.mark.parametrize("B,d,V", [(130, 128, 66308), (300, 1024, 65476)])
def test_probe_of_many_prompts(rgd, B, d, V):
    """Probe steps whose argmax comes from the 256-row tiles' keys (partial last row tile, vocabulary ending inside a
    64-column group), against the same prompts probed 30 at a time.  Every maximum is tied four ways, between lane
    halves (tokens 4 apart) and column halves (256 apart) of a tile: the lowest token wins."""
    t = torch()
    bf, k, P = t.bfloat16, 4, 5
    top, layers = _world(t, B, d, 128, 1, 1, V)
    ids = t.arange(V, device="cuda")
    top["lm_head"] = top["lm_head"][ids & ~(4 | 256)].contiguous()
    g = t.Generator(device="cuda").manual_seed(d)
    pk, pv = t.randn(1, B, 1, P, 128, generator=g, device="cuda").to(bf), t.randn(1, B, 1, 1, 128, 64, generator=g, device="cuda").to(bf)
    last = t.randn(B, V, generator=g, device="cuda")
    m = rgd.Model(rgd.ModelConfig(1, d, 1, 1, 128, 128, V, rgd.DTYPE_BF16, 1e-5, 500000.0, 64), top, layers, B)

    def probe(b0, b1):
        n = b1 - b0
        z = lambda *s: t.zeros(s, dtype=bf, device="cuda")  # noqa: E731
        kv = rgd.KV(m, n, P, n, 16, pk[:, b0:b1], pv[:, b0:b1], z(1, n, 1, 16, 128), z(1, n, 1, 128, 16))
        for b in range(n):
            kv.set_prefix_len(b, P)
        tok, length, event = (t.full(s, -5, dtype=t.int32, device="cuda") for s in ((n, k), (n,), (n,)))
        rgd.probe(m, kv, last[b0:b1], None, n, k, 3, -1, tok, length, event)
        return tok, length, event
    got = probe(0, B)
    lots = [probe(b, min(B, b + 30)) for b in range(0, B, 30)]
    for x, parts in zip(got, zip(*lots)):
        assert t.equal(x, t.cat(parts))
    tok = got[0][:, 1:]
    assert bool(((tok >= 0) & (tok < V) & (tok & (4 | 256) == 0)).all()) and bool((got[1] == k).all())
    assert tok.unique().numel() > B  # prompts differ


@pytest.mark.parametrize("heads,kv_heads", [(32, 8), (6, 2)])
def test_tail_attention_of_many_rows(rgd, heads, kv_heads):
    """Rows of a batch large enough for one-wave tail workgroups against the same rows few at a time (four waves):
    prefixes that end past a split, tails of no, one and several 32-position tiles."""
    t = torch()
    bf = t.bfloat16
    g = t.Generator(device="cuda").manual_seed(heads)
    B, n, P = 2048 // kv_heads // 8, 8, 200
    one = t.ones(128, device="cuda")
    w = lambda *s: (t.randn(*s, generator=g, device="cuda") * 0.02).to(bf)  # noqa: E731
    L = {"wq": w(heads * 128, 128), "wk": w(kv_heads * 128, 128), "wv": w(kv_heads * 128, 128), "wo": w(128, heads * 128),
         "w_gate": w(128, 128), "w_up": w(128, 128), "w_down": w(128, 128), "attn_norm": one, "ffn_norm": one}
    m = rgd.Model(rgd.ModelConfig(1, 128, heads, kv_heads, 128, 128, 128, rgd.DTYPE_BF16, 1e-5, 500000.0, 512),
                  {"embed": w(128, 128), "final_norm": one, "lm_head": w(128, 128)}, [L], B * n)
    R, pages = B * n, 7
    q, k = w(R, heads, 128) * 50, w(B, kv_heads, P, 128) * 50
    v = w(B, kv_heads, (P + 63) // 64, 128, 64)
    tk, tv = w(R * pages, kv_heads, 16, 128) * 50, w(R * pages, kv_heads, 128, 16)
    table = t.randperm(R * pages, generator=g, device="cuda").to(t.int32).view(R, pages)
    prompt = [r // n for r in range(R)]
    plen = [P - 3 * (r % 5) for r in range(R)]
    for tail in (0, 5, 32, 101):
        out, few = t.empty(R, heads * 128, dtype=bf, device="cuda"), t.empty(R, heads * 128, dtype=bf, device="cuda")
        rgd.kernel_attention(m, q, prompt, plen, k, v, B, P, tk, tv, 16, table, pages, tail, out)
        for r in range(0, R, 40):
            e = min(R, r + 40)
            rgd.kernel_attention(m, q[r:e].contiguous(), prompt[r:e], plen[r:e], k, v, B, P, tk, tv, 16,
                                 table[r:e].contiguous(), pages, tail, few[r:e])
        t.cuda.synchronize()
        assert t.isfinite(out.float()).all() and t.equal(out, few), tail


def test_attention_reads_q_in_place_or_from_a_copy(rgd):
    """q at a 2-byte offset, and q that is the output buffer, take the copy; both give the bits of q read in place."""
    t = torch()
    bf = t.bfloat16
    g = t.Generator(device="cuda").manual_seed(3)
    top, layers = _world(t, 3, 1024, 128, 8, 2, 128)
    m = rgd.Model(rgd.ModelConfig(1, 1024, 8, 2, 128, 128, 128, rgd.DTYPE_BF16, 1e-5, 500000.0, 512), top, layers, 9)
    w = lambda *s: t.randn(*s, generator=g, device="cuda").to(bf)  # noqa: E731
    R, P, n = 9, 150, 9 * 8 * 128
    q, k, v = w(R, 8 * 128), w(1, 2, P, 128), w(1, 2, 3, 128, 64)
    tk, tv = w(R, 2, 16, 128), w(R, 2, 128, 16)
    pages = t.arange(R, device="cuda", dtype=t.int32).view(R, 1)

    def run(q, out):
        rgd.kernel_attention(m, q, [0] * R, [P - r for r in range(R)], k, v, 1, P, tk, tv, 16, pages, 1, 7, out)
        t.cuda.synchronize()
        return out
    want = run(q, t.empty_like(q))
    off = t.empty(n + 8, dtype=bf, device="cuda")[1:n + 1].view(R, 8 * 128)
    off.copy_(q)
    both = q.clone()
    assert t.isfinite(want.float()).all()
    assert t.equal(run(off, t.empty_like(q)), want) and t.equal(run(both, both), want)


@pytest.mark.parametrize("V", [4, 1028, 8196])
def test_prompt_logits_at_any_float_offset(rgd, V):
    """The first draw copies the prompts' logits 16 bytes at a time where source and tap allow it, else 4."""
    t = torch()
    g = t.Generator(device="cuda").manual_seed(V)
    top, layers = _world(t, V, 1024, 128, 8, 2, V)
    m = rgd.Model(rgd.ModelConfig(1, 1024, 8, 2, 128, 128, V, rgd.DTYPE_BF16, 1e-5, 500000.0, 64), top, layers, 6)
    z = lambda *s: t.zeros(s, dtype=t.bfloat16, device="cuda")  # noqa: E731
    logits = t.randn(2, V, generator=g, device="cuda")
    got = []
    for src, dst in ((0, 0), (1, 0), (0, 1), (3, 2)):
        kv = rgd.KV(m, 2, 16, 6, 16, z(1, 2, 2, 16, 128), z(1, 2, 2, 1, 128, 64), z(1, 6, 2, 16, 128),
                    z(1, 6, 2, 128, 16))
        last = t.empty(2 * V + 4, device="cuda")[src:src + 2 * V].view(2, V)
        last.copy_(logits)
        tap = t.full((6 * V + 4,), -7.0, device="cuda")
        out = t.empty(2, 3, 1, dtype=t.int32, device="cuda")
        rgd.prefill_kv(m, kv, t.zeros(2, 1, dtype=t.int32, device="cuda"), 0, t.empty(2, V, device="cuda"))
        rgd.sample_continuations(m, kv, last, [0, 1], 3, 1, 1.0, 0.1, t.arange(6, device="cuda"), out,
                                 logits_tap=tap[dst:dst + 6 * V].view(1, 6, V))
        t.cuda.synchronize()
        assert t.equal(tap[dst:dst + 6 * V].view(6, V), logits.repeat_interleave(3, 0))
        assert bool((tap[:dst] == -7.0).all()) and bool((tap[dst + 6 * V:] == -7.0).all())
        got.append(out)
    assert all(t.equal(got[0], o) for o in got)
