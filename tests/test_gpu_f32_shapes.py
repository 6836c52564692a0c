"""fp32 kernels at the edges of their tiles, against the oracle.

The projections multiply 16-wide tiles of rows, columns and k; head sizes,
widths and row counts here leave remainders in each, and one FFN width is not a
multiple of 4 (the general kernel).  Tolerance 1e-5 of each row's largest value,
as for the tiny fp32 decoder (fp32 sums of up to 1100 terms)."""
import numpy as np
import pytest

import synth
from oracle.model import Decoder, KVCache
from tests.gpu_common import rel_err, torch
from tests.test_gpu_kernels import _attn_case, _model

pytestmark = pytest.mark.gpu

BASE = synth.scaled(synth.TINY_FP32, name="f32-shapes", weight_std=0.1)
# d_model, heads, kv heads, head_dim, ffn, vocab
SHAPES = [(36, 3, 1, 8, 52, 68), (40, 5, 5, 16, 50, 260), (260, 8, 1, 32, 1100, 132), (1028, 2, 1, 128, 516, 64)]


@pytest.fixture(scope="module")
def rgd():
    import paper_2607_20791_amd as m
    return m


@pytest.mark.parametrize("prompts,n", [(1, 1), (1, 17), (3, 11), (2, 65)])
@pytest.mark.parametrize("shape", SHAPES)
def test_prefill_and_decode_f32(rgd, shape, prompts, n):
    t = torch()
    from paper_2607_20791_amd import session
    d, hq, hk, D, ffn, V = shape
    steps = 3
    w = synth.scaled(BASE, d_model=d, n_heads=hq, n_kv_heads=hk, head_dim=D, ffn=ffn, vocab=V, n_prompts=prompts,
                     prompt_len=n)
    weights = synth.model_weights(w)
    toks = synth.prompt_tokens(w)
    rows = prompts * n
    m = session.build_model(weights, max_rows=max(rows, prompts), max_pos=n + steps)
    kv = session.alloc_kv(m, w, max_prompts=prompts, max_prefix=n, n_pages=prompts)
    last = t.empty(prompts, V, device="cuda")
    rgd.prefill_kv(m, kv, session.to_device(toks), 0, last)
    forced = synth.forced_history(w, prompts, steps)
    tap = t.empty(steps, prompts, V, device="cuda")
    out = t.empty(prompts, 1, steps, dtype=t.int32, device="cuda")
    rgd.sample_continuations(m, kv, last, list(range(prompts)), 1, steps, 1.0, 0.1,
                             t.arange(prompts, device="cuda"), out, forced=session.to_device(forced), logits_tap=tap)
    got_last, got = last.cpu().numpy(), tap.cpu().numpy()
    dec = Decoder(weights)
    for b in range(prompts):
        cache, tail = KVCache(w.n_layers), KVCache(w.n_layers)
        assert rel_err(got_last[b], dec.prefill(toks[b], cache)).max() <= 1e-5
        for s in range(1, steps):
            ref = dec.decode(int(forced[b, s - 1]), cache, tail)
            assert rel_err(got[s, b], np.asarray(ref)).max() <= 1e-5, (b, s)


# head_dim, heads, kv heads: every head size, one and eight heads per KV head
@pytest.mark.parametrize("D,hq,hk", [(8, 8, 1), (16, 3, 3), (32, 6, 2), (64, 8, 1), (128, 16, 2)])
def test_attention_f32_heads(rgd, D, hq, hk):
    """Splits of 256 positions with rows that end in and before them, V blocks past the row's end, tails of more than one block."""
    w = synth.scaled(BASE, head_dim=D, n_heads=hq, n_kv_heads=hk, d_model=64, ffn=64, vocab=64)
    m = _model(rgd, w, max_rows=64, max_pos=2048)
    for P, tail, plens in [(1, 0, None), (257, 1, [1, 64, 255, 256, 257, 9]), (700, 257, [700, 513, 3, 700, 12, 256]),
                           (70, 600, None)]:
        err = _attn_case(rgd, w, m, 3, 2, P, tail, plens=plens, seed=P + tail)
        assert err.max() <= 1e-5, (P, tail, err.max())


@pytest.mark.parametrize("off", [1, 2])
def test_attention_f32_caches_at_any_float(rgd, off):
    """K and V buffers that start 4 and 8 bytes past a 16-byte boundary give the bits of aligned ones."""
    t = torch()
    w = synth.scaled(BASE, head_dim=32, n_heads=4, n_kv_heads=2, d_model=64, ffn=64, vocab=64)
    m = _model(rgd, w, max_rows=8, max_pos=2048)
    g = t.Generator(device="cuda").manual_seed(off)
    rnd = lambda *s: t.randn(s, generator=g, device="cuda")  # noqa: E731
    R, P, tail, n = 6, 300, 37, 3
    q, bufs = rnd(R, 4 * 32), [rnd(1, 2, P, 32), rnd(1, 2, 5, 32, 64), rnd(R * n, 2, 16, 32), rnd(R * n, 2, 32, 16)]
    pages = t.arange(R * n, device="cuda", dtype=t.int32).view(R, n)

    def run(k, v, tk, tv):
        out = t.empty(R, 4 * 32, device="cuda")
        rgd.kernel_attention(m, q, [0] * R, [P - r for r in range(R)], k, v, 1, P, tk, tv, 16, pages, n, tail, out)
        t.cuda.synchronize()
        return out

    def moved(x):
        y = t.empty(x.numel() + 4, device="cuda")[off:off + x.numel()].view(x.shape)
        return y.copy_(x)
    want = run(*bufs)
    assert t.isfinite(want).all() and t.equal(run(*map(moved, bufs)), want)
