"""The prompt pass's projections on their own against the same products in 64 bits."""
import pytest

from prompt_gemm import CASES, project, project_swiglu

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


# Sums: chains of up to 15 k-steps in the worst case (see the formula at the kernel): 2.5e-7.  SwiGLU's results are stored as hi and lo parts, of bf16 to
# 2^-17 of a value; of fp16 to 2^-22, or 2^-25 where lo is subnormal, behind an exponential of some 2^-21.
@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_every_tile(case, dtype):
    import torch
    swiglu, N, K, M, n_wg, _, pieces, _ = case
    dt = getattr(torch, dtype)
    print(f"case {case} {dtype}", flush=True)
    if swiglu:
        err = project_swiglu(N, K, M, dt, n_wg)
        print(err)
        assert err < (2 ** -17 if dt == torch.bfloat16 else 2 ** -20)
    else:
        err, n = project(N, K, M, dt, 8 * N * M, n_wg)
        print(err)
        assert n == pieces and err < 2.5e-7
