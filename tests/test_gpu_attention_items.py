"""GPU parity of the layer step's attention where its variants change: query rows per kv head (16 and 32 are one and two row
tiles, more take several passes), keys per work item (one to several blocks per wavefront, one or two items per compute
unit), ragged ends of the cache."""
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


def shape(hq, hkv, dh, dtype):
    return synth.ModelShape(f"h{hq}-{hkv}x{dh}-{'f16' if dtype == synth.F16 else 'bf16'}", 1, 64, hq, hkv, dh, 64, 64, 10000.0, (), dtype, False)


# (shape, contexts, rows): with 256 compute units, 40 kv heads have 320 smallest items at 1001 positions (two blocks per
# wavefront), 800 at 2500 (four), 128 kv heads 1280 at 1201 (three, two items per compute unit)
CASES = [(shape(4, 1, 128, synth.BF16), (1, 31, 32, 33, 127, 128, 129, 700), (1, 4, 5, 8)),
         (shape(4, 1, 64, synth.F16), (1, 33, 129), (4, 5, 8)),
         (shape(8, 1, 128, synth.BF16), (2, 130), (1, 2, 3, 5, 8)),
         (shape(3, 1, 64, synth.BF16), (65, 300), (5, 6, 7, 8)),
         (shape(40, 40, 128, synth.BF16), (1001, 2500), (1, 8)),
         (shape(80, 40, 64, synth.F16), (1001, 1300), (8,)),
         (shape(160, 40, 64, synth.BF16), (1001, 2500), (4, 8)),
         (shape(128, 128, 64, synth.BF16), (1201,), (3,)),
         (shape(256, 64, 64, synth.F16), (4100,), (8,))]


@pytest.mark.parametrize("s,ctxs,rows", CASES, ids=lambda x: getattr(x, "name", None))
def test_layer_step_attention(ad, s, ctxs, rows):
    import torch
    w = synth.make_weights(s, seed=2, norm_jitter=0.2)
    # (synthetic weights shrink the attention output's projection by 0.05; here it is to show)
    w["layers.0.wo"] = synth.store_as(synth.as_f32(w["layers.0.wo"]) * 20, s.dtype)
    n = max(ctxs) + 8
    g, o = ad.Model(s, w, max_pos=n), orc.Oracle(s, w, max_pos=n)
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
