"""One projection of the prompt pass on its own: operands in the kernels' layouts, the launcher, and the same product in 64 bits."""
import ctypes as C

from paper_2506_03700_amd import binding


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
