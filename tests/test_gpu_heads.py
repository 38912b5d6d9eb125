"""GPU: the vocabulary pass where its kernel changes: a workgroup's rows are 2, 3 or 4 halves of a 16-row tile (up to 4096, 6144 and
8192 ids on 256 compute units), beyond that whole tiles."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2506_03700_amd import synth
from tolerances import check_rows

pytestmark = pytest.mark.gpu

F32, BF16, F16 = synth.F32, synth.BF16, synth.F16


@pytest.fixture(scope="module")
def ad():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


def shape(V, dtype):
    return synth.ModelShape(f"V{V}", 2, 64, 1, 1, 64, 64, V, 10000.0, (1,), dtype, False)


def pointing_at(w, ids):
    """Rows whose normalised value is the head's row of these ids: each has the largest logit of its row, by far."""
    return torch.from_numpy(np.ascontiguousarray(synth.as_f32(w["lm_head"])[ids] * 50)).to("cuda:0")


@pytest.mark.parametrize("V,dtype", [(300, F32), (300, BF16), (5003, F16), (8192, BF16), (10000, F32), (10000, BF16)], ids=str)
def test_logits_that_are_no_numbers_are_passed_by(ad, V, dtype):
    """The token is the largest of the other logits, wherever in its group of rows the one that is no number lies; the confidence is none
    either."""
    s = shape(V, dtype)
    w = synth.make_weights(s, seed=3)
    best = np.array([3, 13, 16, 47, V // 2 + 1, V // 3, V - 9, V - 1])
    hidden = pointing_at(w, best)
    w["lm_head"] = w["lm_head"].copy()
    bad = sorted({int(r) for b in best for r in (b & ~7, b | 7, b ^ 1, b ^ 4) if r < V} - set(best.tolist()))
    w["lm_head"][bad] = {F32: np.nan, F16: np.nan, BF16: 0x7fc0}[dtype]
    g = ad.Model(s, w, max_pos=8)
    z = g.ad_head_logits(2, hidden).cpu().numpy()
    assert np.array_equal(np.isnan(z), np.broadcast_to(np.isin(np.arange(V), bad), z.shape))
    assert np.array_equal(np.nanargmax(z, axis=1), best)
    for layer in (1, 2):
        for r, b in enumerate(best):
            print(f"case V {V} dtype {dtype} layer {layer} id {b}", flush=True)
            tok, conf = g.ad_exit_head(layer, hidden[r])
            assert tok == b and np.isnan(conf)
    for static in (False, True):
        n, nxt, arg = g.ad_verify(hidden, best[:-1] - 1, static=static)
        assert n == 0 and nxt == best[0] and np.array_equal(arg, best)
        n, nxt, arg = g.ad_verify(hidden, best[:-1], static=static)
        assert n == 7 and nxt == best[7] and np.array_equal(arg, best)
    g.close()


@pytest.mark.parametrize("V,dtype", [(V, t) for V in (4096, 4097, 5003, 6144, 6145, 8192, 8193) for t in (F32, BF16, F16)], ids=str)
def test_logits_and_tokens_at_the_edges_of_the_split(ad, V, dtype):
    """2 (4096 ids), 3 (4097 to 6144), 4 halves of a tile per workgroup, beyond 8192 whole tiles: every logit in its place, and among equal
    ones the lowest id, whether they share 8 rows, a tile, a workgroup (24 ids with 3 halves) or none of these."""
    s = shape(V, dtype)
    w = synth.make_weights(s, seed=11, norm_jitter=0.2)
    w["lm_head"] = w["lm_head"].copy()
    best = np.array([2, 17, 33, 1203, 2407, V - 22, V - 2, 41])
    also = np.array([5, 25, 49, 1212, V - 40, V - 5, V - 1, V // 2 + 3])
    w["lm_head"][also] = w["lm_head"][best]
    hidden = pointing_at(w, best)
    g, o = ad.Model(s, w, max_pos=8), orc.Oracle(s, w, max_pos=8)
    h = hidden.cpu().numpy()
    z = g.ad_head_logits(2, hidden).cpu().numpy()
    for r, b in enumerate(best):
        print(f"case V {V} dtype {dtype} id {b}", flush=True)
        check_rows(dtype, z[r], o.head(-1, h[r], want_logits=True)[3], "logits")
        assert z[r, b] == z[r, also[r]] == z[r].max()
        tok, conf = g.ad_exit_head(1, hidden[r])
        e = np.exp(z[r].astype(np.float64) - z[r].max())
        assert tok == b and abs(conf - e.max() / e.sum()) <= 1e-5
    for static in (False, True):
        n, nxt, arg = g.ad_verify(hidden, best[:-1], static=static)
        assert n == 7 and nxt == best[7] and np.array_equal(arg, best)
        n, nxt, arg = g.ad_verify(hidden, also[:-1], static=static)
        assert n == 0 and nxt == best[0] and np.array_equal(arg, best)
    g.close()


@pytest.mark.parametrize("d,dtype", [(d, F32) for d in (512, 528, 1024, 1040, 2048, 2064, 3072, 3088, 4096, 4112, 5120)] +
                         [(d, t) for d in (64, 512, 528, 1024, 1040) for t in (BF16, F16)], ids=str)
def test_large_vocabularies(ad, d, dtype):
    """The widths where a wavefront's share of the inputs, 2, 4, 8, 12, 16 or 20 operand tiles (16-bit models: 2 or 4), is full, and the
    first of the next."""
    s = synth.ModelShape(f"d{d}", 2, d, 1, 1, 64, 64, 8209, 10000.0, (1,), dtype, False)
    w = synth.make_weights(s, seed=7, norm_jitter=0.2)
    g, o = ad.Model(s, w, max_pos=8), orc.Oracle(s, w, max_pos=8)
    for m in (1, 5, 8):
        print(f"case d {d} dtype {dtype} rows {m}", flush=True)
        h = synth.make_hidden(s, m, m)
        z = g.ad_head_logits(2, torch.from_numpy(h).to("cuda:0")).cpu().numpy()
        for r in range(m):
            check_rows(dtype, z[r], o.head(-1, h[r], want_logits=True)[3], "logits")
    g.close()
