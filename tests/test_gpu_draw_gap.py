"""Draws whose u * W falls into a rise of the fp32 running sum where there is no weight.

The draw's scans add the chunk sums of neighbouring lanes in different orders, so
the running sum can rise by an ulp at a chunk (or 256-logit sub-chunk) that holds
no kept token.  Rows and seeds that hit such a rise are found by a numpy model of
the scans; the draw then has to give the first kept token after it (or the
last one before: the exact running sum is within an ulp of u * W)."""
import numpy as np
import pytest

from oracle import philox
from tests.gpu_common import sample_gpu, seeds_tensor, torch

f32 = np.float32
LOG2E = float(f32(1.4426950408889634))  # temperature at which a logit is the base-2 exponent of its weight
P_MIN = 2.0 ** -23
# span (logits per sum), sums, how many random rows precede the row, the empty sum u * W falls into, seed
CASES = {"chunk-38": (4096, 38, 2, 17, 8796268), "chunk-100": (4096, 100, 2, 58, 1409204),
         "sub-608": (256, 608, 0, 70, 1022410), "sub-512": (256, 512, 0, 48, 5007770)}


def _wave_scan(v):
    v, o = v.astype(f32), 1
    while o < 64:
        v = v + np.concatenate([np.zeros(o, f32), v[:-o]])
        o *= 2
    return v


def _running(span, raw):
    """Running sums and their total as the kernels form them: 64 chunks at a time, or SP sub-chunks per lane."""
    n = len(raw)
    if span == 4096:
        r, off, out = np.zeros(256, f32), f32(0), []
        r[:n] = raw
        for i in range(0, 256, 64):
            v = _wave_scan(r[i:i + 64])
            out.append(v + off)
            off = f32(off + v[63])
        out = np.concatenate(out)[:n]
        return out, out[-1]
    sp = (n + 63) // 64
    r = np.zeros(64 * sp, f32)
    r[:n] = raw
    loc = np.cumsum(r.reshape(64, sp), axis=1, dtype=f32)
    incl = _wave_scan(loc[:, -1])
    excl = np.concatenate([np.zeros(1, f32), incl[:-1]])
    return (excl[:, None] + loc).reshape(-1)[:n], incl[63]


def _row(name):
    """(logits, tokens that may be drawn): half of the sums are empty, the others are spelled out in powers of two,
    so that every order of adding them within a span is exact."""
    span, n, skip, gap, seed = CASES[name]
    rng = np.random.default_rng(n)
    for _ in range(skip + 1):
        units = np.where(rng.random(n) < 0.5, 0, rng.integers(1, 1 << 23, n))
    raw = (units * 2.0 ** -22).astype(f32)
    run, total = _running(span, raw)
    u = float(philox.uniform(seed, 0, 0))
    target = f32(f32(u) * total)
    # the first running sum past u * W belongs to a span without weight
    assert np.flatnonzero(run > target)[0] == gap and raw[gap] == 0 and units.max() >= 1 << 22
    z = np.full(n * span, -1.0e4, f32)
    for c in np.flatnonzero(units):
        bits = [b for b in range(23) if units[c] >> b & 1]
        for i, b in enumerate(bits):
            z[c * span + 7 * i % span + 3] = b - 22
    kept = np.flatnonzero(z > -100)
    at = np.searchsorted(kept, gap * span)
    return z, {int(kept[at - 1]), int(kept[at])}


@pytest.mark.parametrize("name", CASES)
def test_the_seed_draws_into_a_rise_without_weight(name):
    z, tokens = _row(name)
    span, _, _, gap, _ = CASES[name]
    assert all(z[t] > -100 and t // span != gap for t in tokens)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,draws", [(1, 1), (1, 2), (130, 1), (130, 2)])
@pytest.mark.parametrize("name", ["chunk-38", "chunk-100"])
def test_given_logits(name, rows, draws):
    """One draw of one row and of many rows (chunk search by 1024 threads), and several draws (by 256)."""
    import paper_2607_20791_amd as rgd
    z, tokens = _row(name)
    got = sample_gpu(rgd, np.tile(z, (rows, 1)), LOG2E, P_MIN, [CASES[name][4]] * rows, draws=draws)[:, 0]
    assert set(got.tolist()) <= tokens


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["sub-608", "sub-512", "chunk-100"])
def test_first_draw_of_continuations(name):
    """The decode path's draw: sub-chunk sums up to 64 chunks, chunk sums above."""
    import paper_2607_20791_amd as rgd
    t = torch()
    z, tokens = _row(name)
    V, d = z.size, 16
    w = lambda *s: t.zeros(s, device="cuda")  # noqa: E731
    L = {"wq": w(16, d), "wk": w(16, d), "wv": w(16, d), "wo": w(d, 16), "w_gate": w(16, d), "w_up": w(16, d),
         "w_down": w(d, 16), "attn_norm": w(d), "ffn_norm": w(d)}
    m = rgd.Model(rgd.ModelConfig(1, d, 1, 1, 16, 16, V, rgd.DTYPE_F32, 1e-5, 500000.0, 8),
                  {"embed": w(V, d), "final_norm": w(d), "lm_head": w(V, d)}, [L], 2)
    kv = rgd.KV(m, 1, 4, 2, 16, w(1, 1, 1, 4, 16), w(1, 1, 1, 1, 16, 64), w(1, 2, 1, 16, 16), w(1, 2, 1, 16, 16))
    kv.set_prefix_len(0, 1)
    out = t.full((1, 2, 1), -1, dtype=t.int32, device="cuda")
    rgd.sample_continuations(m, kv, t.from_numpy(z).cuda().view(1, V), [0], 2, 1, LOG2E, P_MIN,
                             seeds_tensor([CASES[name][4]] * 2), out)
    t.cuda.synchronize()
    assert set(out.flatten().tolist()) <= tokens
