"""One projection of the prompt pass on its own: operands in the kernels' layouts, the launcher, and the same product in 64 bits."""
import ctypes as C

from paper_2506_03700_amd import binding

# Products that take every kind of tile (0..2 up to 64 tokens; 3..8 above: 2x3, 2x4, 3x3, 3x4, 4x3, 4x4 tiles per wavefront) with rows and tokens left over in
# the last ones, by both epilogues, over 19 to 27 k-steps (more than the copies in flight and no multiple of the steps between two emptyings of an accumulator), over
# more than 128 of them (the other number of steps between emptyings), in several pieces, and with a last round of half tiles:
# (SwiGLU, N, K, tokens, compute units, kind, pieces, half tiles)
CASES = [
    (0, 80, 608, 9, 32, 0, 2, 0), (0, 608, 672, 9, 8, 0, 1, 0), (0, 80, 33056, 9, 256, 0, 8, 0), (0, 848, 608, 9, 8, 1, 1, 0),
    (0, 416, 672, 9, 8, 1, 2, 0), (0, 1808, 4128, 9, 8, 1, 1, 0), (0, 528, 608, 36, 8, 2, 1, 0), (0, 144, 800, 36, 8, 2, 3, 0),
    (0, 1808, 4128, 33, 8, 2, 1, 0), (0, 80, 608, 517, 8, 3, 1, 0), (0, 80, 608, 65, 16, 3, 2, 0), (0, 592, 4128, 258, 8, 3, 1, 0),
    (0, 784, 608, 99, 8, 4, 1, 0), (0, 144, 800, 103, 8, 4, 3, 0), (0, 592, 4128, 298, 8, 4, 1, 0), (0, 560, 608, 135, 8, 5, 1, 0),
    (0, 160, 864, 135, 8, 5, 3, 0), (0, 272, 4192, 299, 8, 5, 1, 0), (0, 1040, 608, 99, 8, 6, 1, 0), (0, 272, 864, 99, 8, 6, 3, 0),
    (0, 272, 4128, 387, 8, 6, 1, 0), (0, 400, 608, 262, 8, 7, 1, 0), (0, 400, 608, 543, 8, 7, 1, 8), (0, 400, 672, 130, 8, 7, 2, 0),
    (0, 1184, 704, 129, 8, 7, 2, 8), (0, 800, 4128, 133, 8, 7, 1, 0), (0, 784, 4192, 645, 8, 7, 1, 8), (0, 784, 608, 194, 8, 8, 1, 0),
    (0, 1168, 672, 196, 8, 8, 2, 8), (0, 800, 704, 290, 8, 8, 1, 8), (0, 400, 704, 193, 8, 8, 2, 0), (0, 784, 4128, 578, 8, 8, 1, 8),
    (0, 400, 4192, 390, 8, 8, 1, 0), (1, 80, 608, 10, 24, 0, 1, 0), (1, 80, 4384, 9, 16, 0, 1, 0), (1, 816, 672, 9, 8, 1, 1, 0),
    (1, 784, 4128, 9, 8, 1, 1, 0), (1, 528, 608, 34, 8, 2, 1, 0), (1, 528, 4128, 34, 8, 2, 1, 0), (1, 80, 608, 66, 24, 3, 1, 0),
    (1, 80, 4128, 70, 24, 3, 1, 0), (1, 544, 608, 97, 8, 4, 1, 0), (1, 528, 4128, 97, 8, 4, 1, 0), (1, 544, 608, 134, 8, 5, 1, 0),
    (1, 1072, 4192, 65, 8, 5, 1, 0), (1, 1040, 608, 97, 8, 6, 1, 0), (1, 1072, 4128, 98, 8, 6, 1, 0), (1, 784, 608, 129, 8, 7, 1, 0),
    (1, 400, 608, 525, 8, 7, 1, 8), (1, 784, 4128, 131, 8, 7, 1, 0), (1, 400, 4128, 533, 8, 7, 1, 8), (1, 400, 608, 409, 8, 8, 1, 0),
    (1, 1040, 704, 211, 8, 8, 1, 4), (1, 784, 4128, 194, 8, 8, 1, 0), (1, 784, 4128, 577, 8, 8, 1, 8)
]


def layout(N, K, M, room, swiglu, n_wg):
    """(kind of tile, pieces, k-steps per piece, workgroups, whole tiles among them, fewest pieces); no GPU."""
    L = binding.sched_test_lib()
    L.ad_prompt_test_layout.argtypes = [C.c_int, C.c_int, C.c_int, C.c_size_t, C.c_int, C.c_int, C.POINTER(C.c_int)]
    L.ad_prompt_test_layout.restype = None
    out = (C.c_int * 6)()
    L.ad_prompt_test_layout(N, K, M, room, int(swiglu), n_wg, out)
    return tuple(out)


class PromptGemm(C.Structure):          # csrc/ad_prompt.h
    _fields_ = [("W", C.c_void_p), ("B", C.c_void_p), ("NT", C.c_int), ("KT", C.c_int), ("N", C.c_int), ("M", C.c_int), ("part", C.c_void_p),
                ("part_floats", C.c_size_t), ("scale", C.c_void_p), ("Bnext", C.c_void_p), ("Bnext_KT", C.c_int), ("f16", C.c_int), ("n_rb", C.c_int),
                ("n_tb", C.c_int), ("n_split", C.c_int), ("k_per", C.c_int), ("n_full", C.c_int)]


def weight_tiles(W):
    """[N, K] -> tiles of 16 rows x 32 inputs: [row tile][k-step][input / 8][row][8]"""
    N, K = W.shape
    return W.view(N // 16, 16, K // 32, 4, 8).permute(0, 2, 3, 1, 4).contiguous()


def token_tiles(X, dtype):
    """[M, K] in fp32 -> tiles of 16 tokens x 32 inputs in two planes, hi and lo, with NaN in the last tile's other tokens, and X as the
    planes hold it, in 64 bits"""
    import torch
    M, K = X.shape
    P = torch.full(((M + 15) // 16 * 16, K), float("nan"), device=X.device)
    P[:M] = X
    hi = P.to(dtype)
    lo = (P - hi.float()).to(dtype)
    tiles = [a.view(-1, 16, K // 32, 4, 8).permute(0, 2, 3, 1, 4) for a in (hi, lo)]
    return torch.stack(tiles, 2).contiguous(), (hi.double() + lo.double())[:M]


def from_token_tiles(T, M):
    """hi + lo of the first M tokens, in 64 bits"""
    t = T.double().sum(2).permute(0, 3, 1, 2, 4)          # [token tile][token][k-step][input / 8][8]
    return t.reshape(t.shape[0] * 16, -1)[:M]


def launch(args, swiglu, n_wg):
    """Returns the number of pieces."""
    import torch
    f = binding.lib()["_ZN2ad18launch_prompt_gemmENS_10PromptGemmEbiPiPv"]
    f.argtypes, f.restype = [PromptGemm, C.c_bool, C.c_int, C.POINTER(C.c_int), C.c_void_p], C.c_int
    pieces = C.c_int(0)
    assert f(args, swiglu, n_wg, None if swiglu else C.byref(pieces), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return pieces.value


def project(N, K, M, dtype, room, n_wg=256, seed=0):
    """A product that stores rows, its pieces added up in order: the relative error (2-norm) and the number of pieces.  Everything of the pieces is
    written, and nothing behind them."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    W = (torch.randn(N, K, generator=g, device="cuda:0") * 0.02).to(dtype)
    T, X = token_tiles(torch.randn(M, K, generator=g, device="cuda:0"), dtype)
    Wt, part = weight_tiles(W), torch.full((room + 4096,), float("nan"), device="cuda:0")
    n = launch(PromptGemm(W=Wt.data_ptr(), B=T.data_ptr(), NT=N // 16, KT=K // 32, N=N, M=M, part=part.data_ptr(), part_floats=room,
                          f16=int(dtype == torch.float16)), False, n_wg)
    p = part[:n * M * N].view(n, M, N)
    assert torch.isnan(part[n * M * N:]).all() and not torch.isnan(p).any()
    y = p[0].clone()
    for i in range(1, n):
        y += p[i]
    e = X @ W.double().t()
    return float((y.double() - e).norm() / e.norm()), n


def project_swiglu(N, K, M, dtype, n_wg=256, seed=0):
    """A product of interleaved gate and up rows, through SwiGLU into operand tiles: the relative error (2-norm).  Nothing but the M tokens' N / 2
    features is written."""
    import torch
    F, KT2 = N // 2, (N // 2 + 31) // 32
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    gate, up = ((torch.randn(F, K, generator=g, device="cuda:0") * 0.05).to(dtype) for _ in range(2))
    T, X = token_tiles(torch.randn(M, K, generator=g, device="cuda:0"), dtype)
    scale = 0.5 + torch.rand(M, generator=g, device="cuda:0")
    Wt = weight_tiles(torch.cat([gate.view(-1, 8, K), up.view(-1, 8, K)], 1).reshape(N, K))
    out = torch.full(((M + 15) // 16, KT2, 2, 4, 16, 8), 7.0, device="cuda:0", dtype=dtype)
    launch(PromptGemm(W=Wt.data_ptr(), B=T.data_ptr(), NT=N // 16, KT=K // 32, N=N, M=M, scale=scale.data_ptr(), Bnext=out.data_ptr(), Bnext_KT=KT2,
                      f16=int(dtype == torch.float16)), True, n_wg)
    y = from_token_tiles(out, out.shape[0] * 16)
    assert (y[M:] == 14).all() and (y[:, F:] == 14).all()
    a, b = (scale.double()[:, None] * (X @ w.double().t()) for w in (gate, up))
    e = torch.nn.functional.silu(a) * b
    return float((y[:M, :F] - e).norm() / e.norm())
