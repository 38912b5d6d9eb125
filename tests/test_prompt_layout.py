"""How the prompt pass lays its projections out (host code alone): the tests of its kernels name the tiles that they run."""
import random

from prompt_gemm import CASES, layout


def test_cases_take_the_tiles_they_name():
    for swiglu, N, K, M, n_wg, kind, pieces, halves in CASES:
        k, n, k_per, grid, full, _ = layout(N, K, M, 8 * N * M, swiglu, n_wg)
        assert (k, n, grid - full) == (kind, pieces, halves), (swiglu, N, K, M, n_wg)
    have = {(swiglu, kind, K // pieces > 128 * 32) for swiglu, _, K, _, _, kind, pieces, _ in CASES}
    assert have >= {(s, k, long) for s in (0, 1) for k in range(9) for long in (False, True)}
    assert {k for s, _, _, _, _, k, n, _ in CASES if n > 1} == set(range(9))
    assert {(s, k, n > 1, K > 128 * 32) for s, _, K, _, _, k, n, h in CASES if h} >= {(s, k, False, long) for s in (0, 1) for k in (7, 8) for long in (False, True)} | {
        (0, k, True, False) for k in (7, 8)}
    for s, N, K, M, *_ in CASES:
        assert (K // 32) % 4 and M % 16 and (N // 16) % 4


def test_pieces_cover_the_inputs_and_fit_the_scratch():
    rng = random.Random(1)
    for _ in range(20000):
        N, K, M = 16 * rng.randint(1, 2000), 16 * rng.randint(1, 1200), rng.randint(1, 1024)
        room = rng.choice([N * M, 2 * N * M, 5 * N * M - 1, 100 * N * M])
        swiglu, n_wg = rng.random() < 0.3, rng.choice([8, 64, 256, 304])
        kind, n, k_per, grid, full, fewest = layout(N, K, M, room, swiglu, n_wg)
        KT = (K + 31) // 32
        assert 1 <= n <= (1 if swiglu else 8) and k_per * n >= KT > k_per * (n - 1) and n * N * M <= room and 0 <= full <= grid
        assert (kind < 3) == (M <= 64)
        if not swiglu and k_per > 128:          # long sums only where the pieces are as many as have room
            blocks = -(-(N // 16) // 8) * -(-M // 128)
            assert n == 8 or blocks * (n + 1) > 2 * n_wg or (n + 1) * N * M > room, (N, K, M, room, n_wg)


def test_shapes_of_the_prompt_tests_take_the_tiles_they_name():
    """The lengths of test_gpu_prompt.py's models (256 compute units; the pass takes all tokens but the last)."""
    R = 1024
    for N, K, swiglu, room, want in (
            (2 * 12312, 96, True, 0, {70: 3, 180: 7, 200: 8, 300: 6, 750: 8}), (2 * 6008, 64, True, 0, {200: 4, 300: 5}),
            (8192, 64, False, R * (2 * 8192 + 64), {300: 3, 400: 4, 600: 6, 750: 7, 1000: 8}), (132 * 64, 64, False, R * 132 * 64, {400: 5})):
        for n, kind in want.items():
            k, _, _, grid, full, _ = layout(N, K, n - 1, room, swiglu, 256)
            assert k == kind and (grid > full) == (n == 750 and swiglu), (N, K, n)
    for n in (97, 98, 193, 194, 300):
        assert layout(2 * 200, 224, n - 1, 0, True, 256)[0] == 3          # 96 tokens per workgroup
