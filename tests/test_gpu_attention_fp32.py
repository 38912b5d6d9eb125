"""GPU parity of the fp32 cache's attention where its split changes: 128 (head_dim 128: 64) cached positions per workgroup, one
workgroup per head up to there, a head's query rows dealt to workgroups while compute units are to spare (all in one, and in two
passes of 32, with 32 kv heads at 1001 positions), ragged ends of the cache."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth
from tolerances import check_kv, check_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


def shape(hq, hkv, dh):
    return synth.ModelShape(f"h{hq}-{hkv}x{dh}-f32", 1, 64, hq, hkv, dh, 64, 64, 10000.0, (), synth.F32, False)


CASES = [(shape(4, 1, 64), (0, 1, 3, 127, 128, 129, 300), (1, 5, 8)),
         (shape(3, 1, 128), (1, 63, 64, 65, 200), (1, 2, 7, 8)),
         (shape(256, 32, 64), (1001,), (8,)),
         (shape(40, 40, 128), (501,), (3,))]


@pytest.mark.parametrize("s,ctxs,rows", CASES, ids=lambda x: getattr(x, "name", None))
def test_layer_step_attention(ad, s, ctxs, rows):
    import torch
    w = synth.make_weights(s, seed=2, norm_jitter=0.2)
    # (synthetic weights shrink the attention output's projection by 0.05; here it is to show)
    w["layers.0.wo"] = synth.store_as(synth.as_f32(w["layers.0.wo"]) * 20, s.dtype)
    n = max(ctxs) + 8
    g, o = ad.Model(s, w, max_pos=n), orc.Oracle(s, w, max_pos=n)
    # positions that no call has filled hold values that are no numbers
    K, V = g.kv_views()
    K.fill_(float("nan"))
    V.fill_(float("nan"))
    k, v = synth.make_kv_prefill(s, 3, 0, max(ctxs))
    g.kv_fill(1, k, v)
    o.kv_write(1, 0, k, v)
    for ctx in sorted(ctxs, reverse=True):           # (a call's rows overwrite positions that a longer context no longer uses)
        for m in rows:
            print(f"case {s.name} context {ctx} rows {m}", flush=True)
            g.kv_set_len(1, ctx)
            o.kv_set_len(1, ctx)
            h = synth.make_hidden(s, 10 * ctx + m, m)
            pos = np.arange(ctx, ctx + m)
            hg = torch.from_numpy(h).to("cuda:0")
            g.ad_layer_step(1, hg, pos)
            ho = o.layer_step(1, h, pos)
            check_rows(s.dtype, hg.cpu().numpy(), ho, f"rows at context {ctx}, {m} rows")
            kg, vg = g.kv_read(1, ctx + m)
            ko, vo = o.kv_read(1, ctx, m)
            check_kv(s.dtype, kg[ctx:], ko, "K")
            check_kv(s.dtype, vg[ctx:], vo, "V")
    g.close()


def test_more_query_rows_than_reciprocals_are_exact_for(ad):
    """40001 query heads on one kv head, 8 rows: three of the 320008 query rows (the last heads of tokens 5, 6 and 7) lie where the rounded-up
    reciprocal of 40001 is one too large.  The output projection sees those heads and the first ones alone."""
    import torch
    G, m, ctx = 40001, 8, 3
    mul = ((1 << 32) + G - 1) // G
    assert [r for r in range(G - 1, m * G, G) if r * mul >> 32 != r // G] == [240005, 280006, 320007]
    s = synth.ModelShape(f"h{G}-1x64-f32", 1, 16, G, 1, 64, 8, 16, 10000.0, (), synth.F32, False)
    w = synth.make_weights(s, seed=8)
    wo = np.zeros_like(w["layers.0.wo"])
    for h in (0, 1, G - 2, G - 1):
        wo[:, h * 64:(h + 1) * 64] = w["layers.0.wo"][:, h * 64:(h + 1) * 64] * 20
    w["layers.0.wo"] = wo
    g, o = ad.Model(s, w, max_pos=ctx + m), orc.Oracle(s, w, max_pos=ctx + m)
    k, v = synth.make_kv_prefill(s, 3, 0, ctx)
    g.kv_fill(1, k, v)
    o.kv_write(1, 0, k, v)
    g.kv_set_len(1, ctx)
    o.kv_set_len(1, ctx)
    h = synth.make_hidden(s, 9, m)
    hg = torch.from_numpy(h).to("cuda:0")
    g.ad_layer_step(1, hg, np.arange(ctx, ctx + m))
    check_rows(s.dtype, hg.cpu().numpy() - h, o.layer_step(1, h, np.arange(ctx, ctx + m)) - h, "what the layer adds")
    g.close()


def test_partials_beyond_32_bit_offsets(ad):
    """8192 query rows on one kv head of 128 dimensions at 262400 positions leave 4100 splits' partials, 17 GB: more floats than 32 bits
    count.  All cached keys are zeros, so every position has the same weight; the values of those in a late split are all there is."""
    import torch
    s = synth.ModelShape("h1024-1x128-f32", 1, 16, 1024, 1, 128, 8, 16, 10000.0, (), synth.F32, False)
    ctx, m, first, n_late = 4100 * 64, 8, 4060 * 64, 64
    assert 4060 * 1024 * m * 130 > 1 << 32
    w = synth.make_weights(s, seed=4)
    w["layers.0.w_down"] = np.zeros_like(w["layers.0.w_down"])
    g = ad.Model(s, w, max_pos=ctx + m)
    K, V = g.kv_views()
    v = (np.random.default_rng(5).standard_normal(128) * 3000).astype(np.float32)
    V[0, 0, :, first:first + n_late] = torch.from_numpy(v).to("cuda:0")[:, None]
    g.kv_set_len(1, ctx)
    h = synth.make_hidden(s, 6, m)
    hg = torch.from_numpy(h).to("cuda:0")
    g.ad_layer_step(1, hg, np.arange(ctx, ctx + m))
    # The call's own rows: their weights are e^score against 1 (scores below 0.1 here) and their values below 1, eight of them
    # against the late split's 64 of thousands: 1e-4 of the attention output at most.
    want = np.tile(v.astype(np.float64) * n_late / ctx, 1024) @ w["layers.0.wo"].astype(np.float64).T
    got = hg.cpu().numpy().astype(np.float64) - h
    assert np.max(np.abs(got - want)) <= 1e-3 * np.max(np.abs(want)), (got, want)
    g.close()
