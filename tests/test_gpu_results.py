"""The calls that return with their results against the ones that only enqueue, through the C ABI: same results, in host memory that is not
pinned, call after call (also past the number after which the stream is waited for all the same) and on another stream."""
import ctypes as C

import numpy as np
import pytest

from paper_2506_03700_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [301, 5000])
def test_results_are_there_when_the_call_returns(vocab):
    import torch
    from paper_2506_03700_amd import binding as ad
    shape = synth.TINY.with_(name="tiny-untied", tied_head=False, vocab=vocab, dtype=synth.BF16)
    g = ad.Model(shape, synth.make_weights(shape, seed=1), max_pos=16)
    L, m = g.L, 4
    pin = torch.zeros(64, dtype=torch.int32).pin_memory()
    rng = np.random.default_rng(0)
    P = lambda a: C.c_void_p(a.ctypes.data)
    D = lambda t: C.c_void_p(t.data_ptr())
    at = lambda i: C.c_void_p(pin.data_ptr() + 4 * i)
    for turn in range(300):
        stream = torch.cuda.Stream() if turn % 64 == 63 else torch.cuda.current_stream()
        with torch.cuda.stream(stream):
            s = C.c_void_p(stream.cuda_stream)
            h = torch.randn(m, shape.d_model, device="cuda:0")
            z, zq = (3 * torch.randn(m, vocab, device="cuda:0") for _ in range(2))
            draft = rng.integers(0, vocab, m - 1, dtype=np.int32)
            u = rng.random(2 * m, dtype=np.float32) * np.float32(0.999)
            got = np.full(16, -7, np.int32)
            calls = [
                (lambda f, a, st: f(g.model, 2, D(h), a(0), a(1), st), L.ad_exit_head, L.ad_exit_head_wait, 2),
                (lambda f, a, st: f(g.model, D(h), P(draft), m, a(0), a(1), a(2), st), L.ad_verify, L.ad_verify_wait, 2 + m),
                (lambda f, a, st: f(g.model, D(z), 0.9, float(u[0]), a(0), a(1), st), L.ad_sample_logits, L.ad_sample_logits_wait, 2),
                (lambda f, a, st: f(g.model, D(z), D(zq), P(draft), m, 0.9, P(u[1:m]), P(u[m:2 * m - 1]), float(u[0]), a(0), a(1), a(2), st),
                 L.ad_verify_sampled, L.ad_verify_sampled_wait, 2 + m - 1)]
            for call, enqueue, wait, n in calls:
                got[:] = -7
                assert call(wait, lambda i: C.c_void_p(got.ctypes.data + 4 * i), s) == ad.AD_OK
                have = got.copy()
                pin.fill_(-7)
                assert call(enqueue, at, s) == ad.AD_OK
                stream.synchronize()
                assert np.array_equal(have[:n], pin.numpy()[:n]) and np.all(have[n:] == -7), (turn, enqueue, have, pin[:n])
    g.close()


@pytest.mark.parametrize("vocab", [300, 2049, 32016])
def test_sampling_in_a_graph(vocab):
    """Captured draws and sampled verifications, replayed over other logits with eager calls in between: the results of the eager calls."""
    import torch
    from paper_2506_03700_amd import binding as ad
    shape = synth.TINY.with_(name="small", tied_head=False, n_layers=1, exit_layers=(), d_model=16, n_q_heads=1, n_kv_heads=1, d_ffn=8,
                             dtype=synth.BF16, vocab=vocab)
    g = ad.Model(shape, synth.make_weights(shape, seed=0), max_pos=8)
    m = 3
    z, zq = torch.zeros(m, vocab, device="cuda:0"), torch.zeros(m - 1, vocab, device="cuda:0")
    out = torch.zeros(16, dtype=torch.int32, device="cuda:0")
    draft, ua, ur = np.array([1, 2], np.int32), np.array([0.5, 0.5], np.float32), np.array([0.3, 0.6], np.float32)
    at = lambda i: C.c_void_p(out.data_ptr() + 4 * i)

    def enqueue():
        s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert g.L.ad_sample_logits(g.model, C.c_void_p(z.data_ptr()), 0.9, 0.4, at(0), at(1), s) == ad.AD_OK
        assert g.L.ad_verify_sampled(g.model, C.c_void_p(z.data_ptr()), C.c_void_p(zq.data_ptr()), C.c_void_p(draft.ctypes.data), m, 0.9,
                                     C.c_void_p(ua.ctypes.data), C.c_void_p(ur.ctypes.data), 0.7, at(2), at(3), at(4), s) == ad.AD_OK
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        enqueue()
    for turn in range(4):
        z.normal_(0, 2)
        zq.copy_(z[:m - 1] if turn % 2 else torch.randn_like(zq))
        out.zero_()
        graph.replay()
        have = out.cpu().numpy()
        out.zero_()
        enqueue()
        assert np.array_equal(have, out.cpu().numpy()), turn
        tok, _ = g.ad_sample_logits(z[0], 0.9, 0.4)
        assert tok == have[0]
    g.close()


def test_sampled_results_from_two_streams_in_turn():
    """Waited-for verifications that accept everything, others that reject, and draws, each on the other stream than the call before, whose rows
    are overwritten there as soon as it returns: the results of the same calls with the device drained between them."""
    import torch
    from paper_2506_03700_amd import binding as ad
    V, m, turns = 32016, 4, 48
    shape = synth.TINY.with_(name="small", tied_head=False, n_layers=1, exit_layers=(), d_model=16, n_q_heads=1, n_kv_heads=1, d_ffn=8,
                             dtype=synth.BF16, vocab=V)
    g = ad.Model(shape, synth.make_weights(shape, seed=0), max_pos=8)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    rows = 2 * torch.randn(turns, m, V, device="cuda:0", generator=gen)
    others = 2 * torch.randn(turns, m - 1, V, device="cuda:0", generator=gen)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    z, zq = torch.empty(m, V, device="cuda:0"), torch.empty(m - 1, V, device="cuda:0")
    torch.cuda.synchronize()

    def results(drain):
        out = []
        for t in range(turns):
            with torch.cuda.stream(streams[t % 2]):
                z.copy_(rows[t])
                zq.copy_(rows[t][:m - 1] if t % 3 else others[t])
                n, tok, ratio = g.ad_verify_sampled(z, zq, [5, 6, 7], 0.9, [0.5] * 3, [0.3] * 3, 0.1 + 0.8 * t / turns)
                assert t % 3 == 0 or n == m - 1
                out.append((n, tok, tuple(ratio)) if t % 4 else (n, tok, tuple(ratio), g.ad_sample_logits(z[0], 0.9, 0.4)))
            if drain:
                torch.cuda.synchronize()
        return out
    assert results(False) == results(True)
    torch.cuda.synchronize()
    g.close()
