"""The prompt pass's projections on their own against the same products in 64 bits."""
import pytest

from prompt_gemm import project

pytestmark = pytest.mark.gpu


# Relative errors of these products with pieces in powers of two, as many as leave a workgroup of 128 x 128 two per compute unit, and chains of up to 8
# k-steps (N, K, tokens, scratch in floats, the error then); with fewer pieces and such chains it was 1.02 to 1.33 times
# that.  An error is an average over all outputs, which repeats itself within 1 % from one set of random operands to the next.
@pytest.mark.parametrize("N,K,M,room,error", [
    (3072, 2048, 16, 1024 * 12288, 1.351e-7), (2048, 2048, 65, 1024 * 12288, 1.308e-7), (2048, 2048, 450, 1024 * 12288, 1.305e-7),
    (1024, 1024, 16, 1024 * 4864, 1.288e-7), (1024, 2816, 65, 1024 * 4096, 1.457e-7), (4096, 4096, 1023, 1024 * 22528, 1.508e-7),
    (4096, 14336, 512, 1024 * 16384, 1.623e-7), (5120, 5120, 700, 1024 * 29184, 1.536e-7), (5120, 13824, 300, 1024 * 25600, 1.620e-7)])
def test_short_chains(N, K, M, room, error):
    import torch
    print(f"case {N} x {K}, {M} tokens", flush=True)
    got, pieces = project(N, K, M, torch.bfloat16, room)
    assert got < 1.01 * error, (got, pieces)
