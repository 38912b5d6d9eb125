"""GPU parity at the widths where the projections over d_model change from one kernel instance to the next (a wavefront's share of
the inputs is 8 operand tiles up to d_model 2048 in 16 bits, 2 up to 512 in fp32): the last width of the narrow instance, whose
share is full, and the first of the next."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth
from tolerances import NEAR_TIE, TOL, check_kv, check_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


WIDTHS = [(synth.BF16, 2048), (synth.BF16, 2064), (synth.F16, 2048), (synth.F16, 2064), (synth.F32, 512), (synth.F32, 528)]


@pytest.mark.parametrize("dtype,d", WIDTHS, ids=[f"{('f32', 'bf16', 'f16')[t]}-{d}" for t, d in WIDTHS])
def test_layers_and_heads_at_the_edges_of_an_instance(ad, dtype, d):
    """The first layer's inputs are normalised by the kernel, the second's come packed from the first; the head takes rows of its own."""
    s = synth.ModelShape(f"d{d}", 3, d, 4, 2, 64, 200, 301, 10000.0, (2,), dtype, False)
    w = synth.make_weights(s, seed=21, norm_jitter=0.2)
    g, o = ad.Model(s, w, max_pos=64), orc.Oracle(s, w, max_pos=64)
    toks = synth.make_prompt(s, 3, 30)
    start = 0
    for m in (1, 8, 3, 5, 2, 8):
        print(f"case d_model {d} dtype {dtype} rows {m}", flush=True)
        pos = np.arange(start, start + m)
        hg, ho = g.ad_embed(toks[start:start + m]), o.embed(toks[start:start + m])
        g.ad_layer_steps(1, 3, hg, pos)
        for l in (1, 2, 3):
            ho = o.layer_step(l, ho, pos)
        check_rows(dtype, hg.cpu().numpy(), ho, f"rows {start}..{start + m - 1}")
        for layer, slot in ((2, 0), (3, -1)):
            z = g.ad_head_logits(layer, hg).cpu().numpy()
            for r in range(m):
                tok, conf, margin, want = o.head(slot, ho[r], want_logits=True)
                check_rows(dtype, z[r], want, f"logits of the head at layer {layer}")
                tok_g, conf_g = g.ad_exit_head(layer, hg[r])
                if margin >= NEAR_TIE:
                    assert tok_g == tok and abs(conf_g - conf) <= 5 * TOL[dtype] * conf
        start += m
    for l in (1, 2, 3):
        (kg, vg), (ko, vo) = g.kv_read(l, start), o.kv_read(l, 0, start)
        check_kv(dtype, kg, ko, f"K of layer {l}")
        check_kv(dtype, vg, vo, f"V of layer {l}")
    g.close()
