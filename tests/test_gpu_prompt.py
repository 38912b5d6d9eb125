"""GPU parity of the prompt pass (many prompt tokens through a layer at once) against the CPU oracle: caches and the
logits that follow, at the edges of its tiles, over several passes, with grouped and ungrouped heads and odd widths."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth
from prompt_gemm import layout
from tolerances import check_kv, check_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


# d_model 208 and d_ffn 200 are no multiples of an operand tile's 32 inputs; 3 query heads per kv head
ODD = synth.TINY.with_(name="odd-bf16", dtype=synth.BF16, tied_head=False, n_q_heads=6, n_kv_heads=2, head_dim=64, d_model=208, d_ffn=200,
                       vocab=301, n_layers=3, exit_layers=(1,), rope_base=500000.0)
DH128 = ODD.with_(name="dh128-bf16", n_q_heads=4, n_kv_heads=1, head_dim=128, d_model=256, d_ffn=688)
MHA = ODD.with_(name="mha-f16", dtype=synth.F16, n_q_heads=3, n_kv_heads=3, head_dim=128, n_layers=2)


def follow_up(shape, g, o, prompt):
    """Both sides take the prompt, then one token more; caches of all layers and that token's logits are compared."""
    n = len(prompt)
    g.ad_generate(prompt, 1, 2.0, 0)
    o.generate_greedy(prompt, 1)
    assert g.kv_lens() == o.kv_lens() == [n] * shape.n_layers
    for l in range(1, shape.n_layers + 1):
        ko, vo = o.kv_read(l, 0, n)
        kg, vg = g.kv_read(l, n)
        check_kv(shape.dtype, kg, ko, f"K of layer {l}, {n} tokens")
        check_kv(shape.dtype, vg, vo, f"V of layer {l}, {n} tokens")
    h, ho = g.ad_embed([7]), o.embed([7])
    for l in range(1, shape.n_layers + 1):
        g.ad_layer_step(l, h, [n])
        ho = o.layer_step(l, ho, np.array([n]))
    check_rows(shape.dtype, h.cpu().numpy(), ho, f"row after {n} tokens")


# the prompt pass takes all but the last token of the prompt: 8 is the most that is left to a layer step; 16, 32, 64, 96, 192, 288 tokens are where
# tiles and, in these shapes, workgroups of tokens of the projections end and the variants change, multiples of 64 rows (21 and a third, 16 and 64
# tokens) those of the attention, 256 tokens those of the other kernels
@pytest.mark.parametrize("shape", [ODD, ODD.with_(name="odd-f16", dtype=synth.F16), DH128, MHA], ids=lambda s: s.name)
def test_prompt_lengths_at_tile_edges(ad, shape):
    w = synth.make_weights(shape, seed=4, norm_jitter=0.2)
    max_pos = 320
    g, o = ad.Model(shape, w, max_pos=max_pos), orc.Oracle(shape, w, max_pos=max_pos)
    for n in (8, 9, 15, 17, 31, 32, 33, 64, 65, 96, 97, 98, 127, 128, 129, 192, 193, 194, 256, 257, 289, 290, 300):
        print(f"case {shape.name} {n} tokens", flush=True)
        follow_up(shape, g, o, synth.make_prompt(shape, n, n + 1))
    g.close()


# Every tile of the projections (128, 192 or 256 rows by 96 or 128 tokens) with rows and tokens left over in the last ones, over two or three k-steps
# (longer contractions: test_gpu_prompt_gemm.py; that the lengths take these tiles: test_prompt_layout.py).  Gate and up:
# 2 x 3 tiles a wavefront at 70 tokens, 4 x 3 at 180, 4 x 4 at 200, 3 x 4 at 300, 4 x 4 and a last round of halves at 750 (and 1000 rows further on, 2 x 4 at
# 200, 3 x 3 at 300); Wo and down of the widest model: 2 x 3 at 300, 2 x 4 at 400, 3 x 4 at 600, 4 x 3 at 750, 4 x 4 at 1000; q/k/v of
# 130 heads: 3 x 3 at 400.
@pytest.mark.parametrize("shape,lengths", [
    (ODD.with_(name="ffn-12312", d_model=96, d_ffn=12312, n_layers=2), (70, 180, 200, 300, 750)),
    (ODD.with_(name="ffn-6008-f16", dtype=synth.F16, d_model=64, d_ffn=6008, n_layers=2), (200, 300)),
    (ODD.with_(name="wide", d_model=8192, d_ffn=64, n_q_heads=1, n_kv_heads=1, n_layers=2), (300, 400, 600, 750, 1000)),
    (ODD.with_(name="heads-130", d_model=64, n_q_heads=130, n_kv_heads=1, n_layers=2), (400,))], ids=lambda x: getattr(x, "name", ""))
def test_every_tile_of_the_projections(ad, shape, lengths):
    w = synth.make_weights(shape, seed=4, norm_jitter=0.2)
    g, o = ad.Model(shape, w, max_pos=1024), orc.Oracle(shape, w, max_pos=1024)
    for n in lengths:
        print(f"case {shape.name} {n} tokens", flush=True)
        follow_up(shape, g, o, synth.make_prompt(shape, n, n + 1))
    g.close()


# beyond 1024 tokens: a second pass at position 1024, of more and of fewer tokens than a layer step takes
@pytest.mark.parametrize("shape,n", [(DH128, 1024), (DH128, 1031), (ODD, 1100)], ids=["one-pass", "pass-and-step", "two-passes"])
def test_prompts_longer_than_a_pass(ad, shape, n):
    w = synth.make_weights(shape, seed=5, norm_jitter=0.2)
    g, o = ad.Model(shape, w, max_pos=1152), orc.Oracle(shape, w, max_pos=1152)
    follow_up(shape, g, o, synth.make_prompt(shape, n, n + 1))
    g.close()


def test_storage_without_the_scratch_is_a_cache_too(ad):
    """ad_kv_create takes storage that ends before the prompt pass's scratch: the same caches, by layer steps."""
    import torch
    shape = DH128
    w = synth.make_weights(shape, seed=6, norm_jitter=0.2)
    g, o = ad.Model(shape, w, max_pos=200), orc.Oracle(shape, w, max_pos=200)
    L, full = g.L, g.L.ad_kv_bytes(C.byref(g.cfg), 200)
    kv, stream = C.c_void_p(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.ad_kv_create(g.model, C.c_void_p(g.kv_storage.data_ptr()), 4096, 200, stream, C.byref(kv)) == ad.AD_ENOMEM
    L.ad_kv_destroy(g.kv)
    assert L.ad_kv_create(g.model, C.c_void_p(g.kv_storage.data_ptr()), full - 256, 200, stream, C.byref(kv)) == ad.AD_OK
    g.kv = kv
    follow_up(shape, g, o, synth.make_prompt(shape, 1, 71))
    g.close()


# The pieces of q/k/v (N 1536) and Wo (N 2048) of some 100 tokens, five or four and three of them, take 2.4 to 3 MB: more than the 2 MB set aside for
# them in a cache of 128 rows, so that they run on into the SwiGLU activations; those of down lie over queries and attention output.
SHARED = ODD.with_(name="shared-bf16", n_q_heads=16, n_kv_heads=4, d_model=2048, d_ffn=2752)


def same_bits_in_poisoned_storage(ad, shape, max_pos, lengths):
    import torch
    w = synth.make_weights(shape, seed=8, norm_jitter=0.2)
    g = ad.Model(shape, w, max_pos=max_pos)
    want = []
    for fill in (0, 255):
        g.L.ad_kv_destroy(g.kv)
        g.kv_storage.fill_(fill)
        kv = C.c_void_p()
        assert g.L.ad_kv_create(g.model, C.c_void_p(g.kv_storage.data_ptr()), g.kv_storage.numel(), max_pos,
                                C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(kv)) == ad.AD_OK
        g.kv = kv
        for i, n in enumerate(lengths):
            g.ad_generate(synth.make_prompt(shape, n, n), 3, 2.0, 0)
            got = [a for l in range(1, shape.n_layers + 1) for a in g.kv_read(l, n)]
            if fill == 0:
                want.append(got)
            assert all(np.array_equal(a, b) and np.all(np.isfinite(a)) for a, b in zip(got, want[i])), (fill, n)
    g.close()


@pytest.mark.parametrize("shape", [ODD, ODD.with_(name="odd-f16", dtype=synth.F16), DH128, MHA], ids=lambda s: s.name)
def test_nothing_is_read_that_was_not_written(ad, shape):
    """A cache in storage full of NaN gives the same bits as one in zeros, prompt after prompt."""
    same_bits_in_poisoned_storage(ad, shape, 320, (17, 10, 140, 70, 300))


@pytest.mark.parametrize("shape", [SHARED, SHARED.with_(name="shared-f16", dtype=synth.F16)], ids=lambda s: s.name)
def test_pieces_in_scratch_of_other_steps(ad, shape):
    import torch
    own, room = 128 * 2 * shape.d_model, 128 * (2 * shape.d_model + shape.d_ffn)        # floats
    for N, K in ((shape.d_q + 2 * shape.d_kv, shape.d_model), (shape.d_model, shape.d_q)):
        for m in (99, 109, 116):
            pieces = layout(N, K, m, room, False, torch.cuda.get_device_properties(0).multi_processor_count)[1]
            assert own < pieces * m * N <= room
    same_bits_in_poisoned_storage(ad, shape, 120, (100, 10, 65, 110))
    w = synth.make_weights(shape, seed=9, norm_jitter=0.2)
    g, o = ad.Model(shape, w, max_pos=120), orc.Oracle(shape, w, max_pos=120)
    for n in (34, 100, 117):
        print(f"case {shape.name} {n} tokens", flush=True)
        follow_up(shape, g, o, synth.make_prompt(shape, n, n + 1))
    g.close()


def test_activations_of_four_gigabytes(ad):
    """1024 tokens' inputs to the down projection would take 4.5 GB: fewer tokens to a pass, and the same caches as by layer steps
    (the last tokens of a pass are the ones whose tiles lie furthest)."""
    shape = synth.TINY.with_(name="wide-ffn", dtype=synth.BF16, tied_head=False, n_q_heads=1, n_kv_heads=1, d_model=16, d_ffn=1100000, vocab=64,
                             n_layers=2, exit_layers=())
    w = synth.make_weights(shape, seed=7)
    # (the sums over 1.1 million inputs are to show next to the residual, and not to drown it)
    w["layers.0.w_down"] = synth.store_as(synth.as_f32(w["layers.0.w_down"]) * 20, shape.dtype)
    n, m = 1024, 8
    g = ad.Model(shape, w, max_pos=n + 8)
    prompt = synth.make_prompt(shape, 2, n)
    g.ad_generate(prompt, 1, 2.0, 0)
    k, v = g.kv_read(2, n)
    g.kv_truncate(0)
    for s in range(0, n, m):
        h = g.ad_embed(prompt[s:s + m])
        g.ad_layer_steps(1, 2, h, np.arange(s, s + m))
    k0, v0 = g.kv_read(2, n)
    check_kv(shape.dtype, k, k0, "K of layer 2")
    check_kv(shape.dtype, v, v0, "V of layer 2")
    g.close()
