"""GPU: models made one after the other in the same memory."""
import pytest

from oracle import oracle as orc
from paper_2506_03700_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_03700_amd import binding
    binding.lib()
    return binding


def test_a_new_model_does_not_see_an_earlier_ones_results(ad):
    """Models made one after the other get the same pinned words: the first evaluation of each waits for its own result.  Every
    model has a prompt of its own, and each one's token differs from the one before, so a word left over is a wrong answer."""
    shape = synth.TINY.with_(name="tiny-untied", tied_head=False, vocab=512)
    w = synth.make_weights(shape, seed=1)
    o = orc.Oracle(shape, w, max_pos=64)
    cases = []
    for seed in range(1, 100):
        prompt = synth.make_prompt(shape, seed, 20)
        tok, margin = o.generate_greedy(prompt, 1)
        if margin[0] > 1e-2 and (not cases or tok[0] != cases[-1][1]):
            cases.append((prompt, tok[0]))
        if len(cases) == 6:
            break
    assert len(cases) == 6
    for i, (prompt, want) in enumerate(cases):
        g = ad.Model(shape, w, max_pos=64)
        out, _, _ = g.ad_generate(prompt, 1, 2.0, 0)
        assert out[0] == want, i
        g.close()
