"""GPU: draws and sampled verification at the edges of the segments a logits row is cut into (of equal length, at most 2048 ids, but no
more than 512 of them: longer ones beyond 1 048 576 ids), with masked ids and masked segments, against the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth

pytestmark = pytest.mark.gpu

SMALL = synth.TINY.with_(name="small", tied_head=False, n_layers=1, exit_layers=(), d_model=16, n_q_heads=1, n_kv_heads=1, d_ffn=8, dtype=synth.BF16)


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


def segment_length(V):
    n = min(-(-V // 2048), 512)
    return -(-V // n)


# 2049: two segments of 1025 and 1024 ids; 4097: three of 1366; 600001: 293 of 2048; 1100003: 512 of 2149, more than a thread keeps
@pytest.mark.parametrize("V", [1, 2047, 2048, 2049, 4097, 600001, 1100003])
def test_draws_and_verification_at_segment_edges(ad, V):
    import torch
    seg = segment_length(V)
    g = ad.Model(SMALL.with_(vocab=V), synth.make_weights(SMALL.with_(vocab=V), seed=0), max_pos=8)
    rng = np.random.default_rng(V)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    last = (V - 1) // seg * seg              # the last segment's first id
    edges = sorted({t for t in (0, 1, seg - 1, seg, seg + 1, last - 1, last, V - 2, V - 1) if 0 <= t < V})
    for t in edges:
        print(f"case V={V} token {t}", flush=True)
        z = (rng.standard_normal(V) * 0.5).astype(np.float32)
        z[t] = 16.0
        p = orc.softmax_t(z.astype(np.float64), 1.0)
        u = float(np.float32(p[:t].sum() + p[t] / 2))
        tok, prob = g.ad_sample_logits(dev(z), 1.0, u)
        assert tok == t == orc.sample_cdf(p, u)[0] and abs(prob - p[t]) <= 1e-5 * p[t]
        # only t and the edges have any weight, whatever the draw; masked ids are never drawn
        z = np.full(V, -np.inf, dtype=np.float32)
        z[edges] = rng.standard_normal(len(edges)).astype(np.float32)
        p = orc.softmax_t(z.astype(np.float64), 1.0)
        for u in (0.0, float(np.float32(rng.random())), float(np.float32(1 - 2.0 ** -24))):
            tok, prob = g.ad_sample_logits(dev(z), 1.0, u)
            want, margin = orc.sample_cdf(p, u)
            assert tok in edges and abs(prob - p[tok]) <= 1e-5 * p[tok]
            assert tok == want or margin < 1e-6
        # a rejected draft: p* exceeds p_draft by far at t, and little or nowhere else; then at all the edges
        for more in ((), edges) if V > 1 else ():
            zf = (rng.standard_normal((2, V)) * 0.5).astype(np.float32)
            zq = zf[:1].copy()
            d = edges[0] if t != edges[0] else edges[-1]
            zf[0, list(more)] = 12.0 + rng.random(len(more)).astype(np.float32)
            zf[0, t] = 14.0
            zf[0, d] = zq[0, d]
            zq[0, d] = 14.0
            ur = float(np.float32(rng.random()))
            n, nxt, ratio = g.ad_verify_sampled(dev(zf), dev(zq), [d], 1.0, [0.5], [ur], 0.5)
            p, q = orc.softmax_t(zf[0].astype(np.float64), 1.0), orc.softmax_t(zq[0].astype(np.float64), 1.0)
            acc, want, _, margin = orc.accept_or_resample(p, q, d, 0.5, ur)
            assert n == 0 and not acc and abs(ratio[0] - p[d] / q[d]) <= 1e-4 * p[d] / q[d]
            # (fp32 sums of V weights: the draw may fall to the other side of a boundary it is this close to)
            assert nxt == want or margin < 1e-5
    # the spread of a real row: draws all over it, then with one of its segments masked
    for u in rng.random(6).astype(np.float32):
        z = (rng.standard_normal(V) * 0.5).astype(np.float32)
        s = int(rng.integers(0, (V - 1) // seg + 1))
        for masked in (0, seg):
            if masked and V <= seg:
                continue
            z[s * seg:s * seg + masked] = -np.inf
            p = orc.softmax_t(z.astype(np.float64), 1.0)
            tok, prob = g.ad_sample_logits(dev(z), 1.0, float(u))
            want, margin = orc.sample_cdf(p, float(u))
            # (the target may fall between neighbours of about 1 / V each: the drawn id's own share and no more lies between)
            assert p[min(tok, want):max(tok, want) + 1].sum() <= p[tok] + p[want] + 1e-5 and abs(prob - p[tok]) <= 1e-5 * p[tok]
    g.close()


@pytest.mark.parametrize("V", [301, 2047, 2048, 2049])
def test_rows_of_one_segment_and_of_two(ad, V):
    """Rows of one segment, up to four and more (whose statistics come from the last kernel, from one of their own), and of two: no
    draft rejected, the first, one in the middle, the last."""
    import torch
    g = ad.Model(SMALL.with_(vocab=V), synth.make_weights(SMALL.with_(vocab=V), seed=0), max_pos=8)
    rng = np.random.default_rng(V)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    for m in (1, 2, 4, 5, 8):
        for bad in sorted({None, 0, (m - 1) // 2, m - 2} if m > 1 else {None}, key=str):
            print(f"case V={V} m={m} rejected {bad}", flush=True)
            zf = rng.standard_normal((m, V)).astype(np.float32)
            zq = (zf[:m - 1] + 0.1 * rng.standard_normal((m - 1, V))).astype(np.float32)
            draft = rng.integers(0, V, m - 1).astype(np.int32)
            if bad is not None:
                zq[bad, draft[bad]] += 12.0
            ur, uf = rng.random(m - 1).astype(np.float32), float(np.float32(rng.random()))
            n, nxt, ratio = g.ad_verify_sampled(dev(zf), dev(zq) if m > 1 else None, draft, 0.7, np.full(m - 1, 0.3, np.float32), ur, uf)
            assert n == (m - 1 if bad is None else bad)
            p = lambda z: orc.softmax_t(z.astype(np.float64), 0.7)
            for k in range(m - 1):
                want = p(zf[k])[draft[k]] / p(zq[k])[draft[k]] if k <= n else 0.0
                assert abs(ratio[k] - want) <= 1e-5 * want
            if bad is None:
                want, margin = orc.sample_cdf(p(zf[n]), uf)
            else:
                _, want, _, margin = orc.accept_or_resample(p(zf[n]), p(zq[n]), int(draft[n]), 0.3, float(ur[n]))
            # (fp32 sums of V weights in another order: the draw may fall to the other side of a boundary it is this close to)
            assert nxt == want or margin < 1e-5
    g.close()


@pytest.mark.parametrize("V", [2049, 8192])
def test_a_segment_that_is_not_a_number_shows(ad, V):
    """A row's sum is no number if one of its logits is none, also where a whole segment consists of such values."""
    import torch
    seg = segment_length(V)
    n_seg = -(-V // seg)
    g = ad.Model(SMALL.with_(vocab=V), synth.make_weights(SMALL.with_(vocab=V), seed=0), max_pos=8)
    rng = np.random.default_rng(V)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    for s in range(n_seg):
        for bad in (slice(s * seg, (s + 1) * seg), slice(s * seg, s * seg + 1)):
            z = rng.standard_normal((3, V)).astype(np.float32)
            z[0, bad] = np.nan
            z[0, s * seg + 1] = -np.inf          # and a masked id among them
            tok, prob = g.ad_sample_logits(dev(z[0]), 0.8, 0.5)
            assert np.isnan(prob) and tok == np.flatnonzero(np.isfinite(z[0]))[-1]
            d = V - 1 if s == 0 else 0
            n, nxt, ratio = g.ad_verify_sampled(dev(z[:2]), dev(z[2:]), [d], 0.8, [0.5], [0.5], 0.5)
            assert np.isnan(ratio[0])
    g.close()
