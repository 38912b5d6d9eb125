"""GPU: models made one after the other in the same memory."""
import pytest

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
    """Models made one after the other get the same pinned words: the first evaluation of each waits for its own result."""
    shape = synth.TINY.with_(name="tiny-untied", tied_head=False, vocab=512)
    w = synth.make_weights(shape, seed=1)
    first = None
    for i in range(4):
        g = ad.Model(shape, w, max_pos=64)
        out, _, _ = g.ad_generate(synth.make_prompt(shape, 1, 20), 1, 2.0, 0)
        first = out[0] if first is None else first
        assert out[0] == first, i
        g.close()
