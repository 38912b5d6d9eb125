"""GPU parity of the projections with few row tiles per workgroup, at the shapes where their split changes: a workgroup's rows are 2,
3 or 4 halves of a 16-row tile (256, 257 and 385 tiles and more on 256 compute units), the contraction has an odd number of k-steps or fewer
than there are wavefronts, the inputs end inside a k-step, the rows end inside a workgroup's share."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth
from tolerances import check_kv, check_rows

pytestmark = pytest.mark.gpu

F32, BF16, F16 = synth.F32, synth.BF16, synth.F16

# (name, d_model, query heads, kv heads, head_dim, d_ffn): tiles of q/k/v, Wo and down, gate/up
SHAPES = [
    ("d272-qkv385", 272, 32, 8, 128, 88),        # 384, 17, 11; 9 k-steps, the last one half filled
    ("d48-qkv513", 48, 64, 2, 128, 2056),        # 544 (another kernel), 3, 257; 2 k-steps for 8 wavefronts
    ("d112-qkv400", 112, 46, 2, 128, 4088),      # 400, 7, 511; down has 128 k-steps
    ("d4112", 4112, 2, 1, 64, 200),              # 16, 257, 25; 129 k-steps
]
WIDE = [("d6160", 6160, 2, 2, 64, 72), ("d8192", 8192, 2, 1, 64, 40)]          # 385 and 512 tiles of Wo and down
CASES = [(s, t) for s in SHAPES for t in (F32, BF16, F16)] + [(s, t) for s in WIDE for t in (BF16, F16)]


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("shape,dtype", CASES, ids=[f"{s[0]}-{('f32', 'bf16', 'f16')[t]}" for s, t in CASES])
def test_layers_at_the_edges_of_the_split(ad, shape, dtype):
    """Two layers: the first projects rows that it normalises itself, the second takes them packed from the first."""
    name, d, hq, hkv, dh, f = shape
    s = synth.ModelShape(name, 2, d, hq, hkv, dh, f, 64, 10000.0, (1,), dtype, False)
    w = synth.make_weights(s, seed=5, norm_jitter=0.2)
    g, o = ad.Model(s, w, max_pos=64), orc.Oracle(s, w, max_pos=64)
    toks = synth.make_prompt(s, 1, 12)
    start = 0
    for m in (1, 8, 3):
        print(f"case {name} dtype {dtype} rows {m}", flush=True)
        pos = np.arange(start, start + m)
        hg, ho = g.ad_embed(toks[start:start + m]), o.embed(toks[start:start + m])
        g.ad_layer_steps(1, 2, hg, pos)
        for l in (1, 2):
            ho = o.layer_step(l, ho, pos)
        check_rows(dtype, hg.cpu().numpy(), ho, f"rows {start}..{start + m - 1}")
        start += m
    for l in (1, 2):
        (kg, vg), (ko, vo) = g.kv_read(l, start), o.kv_read(l, 0, start)
        check_kv(dtype, kg, ko, f"K of layer {l}")
        check_kv(dtype, vg, vo, f"V of layer {l}")
    g.close()


@pytest.mark.parametrize("d,dtype", [(272, BF16), (4096, F16), (4112, BF16), (1024, F32), (1040, F32)], ids=str)
def test_exit_head_transform(ad, d, dtype):
    """The transform of an exit head: rows normalised, multiplied, packed; up to 128 (fp32: 32) k-steps, and beyond."""
    s = synth.ModelShape(f"t{d}", 2, d, 2, 1, 64, 64, 300, 10000.0, (1,), dtype, False)
    w = synth.make_weights(s, seed=6, norm_jitter=0.2, with_T=True)
    g, o = ad.Model(s, w, max_pos=8), orc.Oracle(s, w, max_pos=8)
    toks = synth.make_prompt(s, 2, 8)
    for m in (1, 5, 8):
        print(f"case transform d {d} dtype {dtype} rows {m}", flush=True)
        hg, ho = g.ad_embed(toks[:m]), o.embed(toks[:m])
        z = g.ad_head_logits(1, hg).cpu().numpy()
        for r in range(m):
            check_rows(dtype, z[r], o.head(0, ho[r], want_logits=True)[3], "logits")
    g.close()
