"""GPU parity of attention where scores overflow to minus infinity: such a key has no weight, whether it is alone in its block, fills
a wavefront's blocks, a whole work item or the call's own rows, in the layer step and in the prompt pass."""
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


def lone(shape, rows, in_dim, value, base=None):
    """Every head's last dimension (the slowest to rotate) reads input in_dim alone, with weight `value`; its partner in the
    rotation reads nothing."""
    w = np.zeros((rows, shape.d_model), np.float32) if base is None else synth.as_f32(base).copy()
    for h in range(rows // shape.head_dim):
        w[h * shape.head_dim + shape.head_dim - 1] = w[h * shape.head_dim + shape.head_dim // 2 - 1] = 0.0
        w[h * shape.head_dim + shape.head_dim - 1, in_dim] = value
    return synth.store_as(w, shape.dtype)


def shape(hq, hkv, dh):
    return synth.ModelShape(f"h{hq}-{hkv}x{dh}", 1, 64, hq, hkv, dh, 64, 64, 500000.0, (), synth.BF16, False)


# a query's last dimension is about 100, times 1 / sqrt(dh): against -3e38 in a cache entry the score is below the smallest fp32
BIG = -3e38
# (shape, context, keys that overflow, the call's own keys overflow too): the 33rd key alone in its block; a wavefront's first
# block; all its blocks (256 positions are one item of two blocks per wavefront); the second item of three; the only item's
# own rows beside one cached key; the second of five items of four blocks per wavefront (two row tiles per wavefront)
CASES = [(shape(4, 1, 128), 33, [range(32, 33)], False), (shape(4, 1, 64), 128, [range(32)], False),
         (shape(4, 2, 128), 256, [range(32), range(128, 160)], False), (shape(4, 1, 128), 300, [range(128, 256)], False),
         (shape(8, 1, 64), 1, [], True), (shape(160, 40, 64), 2500, [range(512, 1024)], False)]


@pytest.mark.parametrize("s,ctx,keys,own", CASES, ids=lambda x: getattr(x, "name", None))
def test_layer_step(ad, s, ctx, keys, own):
    import torch
    w = synth.make_weights(s, seed=2)
    w["layers.0.wq"] = lone(s, s.d_q, 0, 30.0, w["layers.0.wq"])
    if own:
        w["layers.0.wk"] = lone(s, s.d_kv, 0, -3e37, w["layers.0.wk"])
    w["layers.0.wo"] = synth.store_as(synth.as_f32(w["layers.0.wo"]) * 20, s.dtype)
    g, o = ad.Model(s, w, max_pos=ctx + 8), orc.Oracle(s, w, max_pos=ctx + 8)
    k, v = synth.make_kv_prefill(s, 3, 0, ctx)
    k = np.array(k)
    k[..., s.head_dim - 1] = 0
    for r in keys:
        k[r.start:r.stop, ..., s.head_dim - 1] = BIG
    k = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(k)).reshape(k.shape)
    g.kv_fill(1, k, v)
    o.kv_write(1, 0, k, v)
    for m in (1, 4, 5, 8):
        print(f"case {s.name} context {ctx} rows {m}", flush=True)
        g.kv_set_len(1, ctx)
        o.kv_set_len(1, ctx)
        h = synth.make_hidden(s, 10 * ctx + m, m)
        h[:, 0] = 4.0
        hg = torch.from_numpy(h).to("cuda:0")
        g.ad_layer_step(1, hg, np.arange(ctx, ctx + m))
        ho = o.layer_step(1, h, np.arange(ctx, ctx + m))
        check_rows(s.dtype, hg.cpu().numpy(), ho, f"rows at context {ctx}, {m} rows")
    g.close()


@pytest.mark.parametrize("n_first,n", [(32, 40), (32, 90), (64, 200)])
def test_prompt(ad, n_first, n):
    """Tokens of a first kind make keys against which the queries of the second kind, and theirs alone, overflow."""
    s = synth.TINY.with_(name="two-kinds", dtype=synth.BF16, tied_head=False, n_q_heads=4, n_kv_heads=1, head_dim=128, d_model=64, d_ffn=64,
                         vocab=128, n_layers=2, exit_layers=(), rope_base=500000.0)
    w = synth.make_weights(s, seed=6)
    w["layers.0.wq"] = lone(s, s.d_q, 1, 30.0, w["layers.0.wq"])
    w["layers.0.wk"] = lone(s, s.d_kv, 0, -3e37, w["layers.0.wk"])
    e = synth.as_f32(w["embed"]).copy() * 20
    e[:64, :2], e[64:, :2] = (4.0, 0.0), (0.0, 4.0)
    w["embed"] = synth.store_as(e, s.dtype)
    rng = np.random.default_rng(n)
    prompt = np.concatenate([rng.integers(0, 64, n_first), rng.integers(64, 128, n - n_first)]).astype(np.int32)
    g, o = ad.Model(s, w, max_pos=256), orc.Oracle(s, w, max_pos=256)
    g.ad_generate(prompt, 1, 2.0, 0)
    o.generate_greedy(prompt, 1)
    for l in (1, 2):
        (kg, vg), (ko, vo) = g.kv_read(l, n), o.kv_read(l, 0, n)
        # (the entries near -1e38 would hide all others in a bound relative to the largest)
        rest = slice(0, s.head_dim - 1) if l == 1 else slice(None)
        check_kv(s.dtype, kg[..., rest], np.reshape(ko, kg.shape)[..., rest], f"K of layer {l}")
        check_kv(s.dtype, vg, np.reshape(vo, vg.shape), f"V of layer {l}")
    g.close()
