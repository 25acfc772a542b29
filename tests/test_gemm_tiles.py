"""The GEMM kernels at the edges of their tiles.  `CASES`: row classes and column remainders through clover_op_gemm, and the
few-output fp32 kernel at one row, one column, K tails and the tile count where the larger tiles take over.  `PLAIN` and
`SWIGLU`: every form (tile, one or several row tiles) of the MFMA kernel, each with fewer stages of K than buffers and with
more, odd stage counts, first and last rows of a row block; the form is asserted, so that another choice by the rule shows.
CB counts 32 columns, 3.5 of them are the tiles of seven blocks.  (The plain result with RB 5 and several row tiles needs more
rows than the operator takes; its loop is that of the SwiGLU cases of that form.)"""
import ctypes as C

import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu

# (path, dtype, M, N, K): path 7 sums K ranges, path 3 writes the whole K's result directly
CASES = [(7, 1, m, n, k) for m in (1, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 256)
         for n, k in ((16, 128), (1040, 640), (400, 4096))]
CASES += [(3, 1, m, n, 512) for m in (1, 31, 64, 65, 128) for n in (48, 2064)]
CASES += [(0, d, m, n, k) for d in (0, 1) for m, n, k in ((1, 1, 4), (17, 5, 260), (16, 257, 256), (33, 1023, 688), (3, 130, 1028))]
# column counts at which the rule takes tiles of 96 columns (6 blocks of 16 fill more of the chip than 8)
CASES += [(7, 1, m, 6144, 4096) for m in (33, 64, 80)] + [(3, 1, m, 22016, 512) for m in (23, 64, 96)]
# 255 tiles of 64 x 64 (the few-output kernel) and 256 (the tiles)
CASES += [(0, 0, 64, 255 * 64, 64), (0, 0, 64, 256 * 64, 64)]


@pytest.mark.parametrize("path,dtype,M,N,K", CASES)
def test_gemm_tile_edges(path, dtype, M, N, K):
    import torch
    print(f"gemm path={path} dtype={dtype} M={M} N={N} K={K}", flush=True)
    lib = clover.load_library()
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    X = rng.standard_normal((M, K)).astype(np.float32)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    if dtype == 1:
        Wb = synth.f32_to_bf16_bits(W)
        Wf = synth.bf16_bits_to_f32(Wb).astype(np.float64)
        Wd = torch.from_numpy(Wb.view(np.int16)).cuda()
    else:
        Wf = W.astype(np.float64)
        Wd = torch.from_numpy(W).cuda()
    Xd = torch.from_numpy(X).cuda()
    ldy = N + 4 - N % 4
    Y = torch.full((M, ldy), -7.0, dtype=torch.float32, device="cuda")
    nb = lib.clover_op_gemm_scratch_bytes(M, N, K)
    # all-NaN scratch: rows that pad the last row block, and whatever a launch leaves unwritten, must not reach a result
    scratch = torch.full((nb,), 255, dtype=torch.uint8, device="cuda")
    rc = lib.clover_op_gemm(path, dtype, C.c_void_p(Xd.data_ptr()), C.c_void_p(Wd.data_ptr()), C.c_void_p(Y.data_ptr()), ldy,
                            M, N, K, C.c_void_p(scratch.data_ptr()), nb, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lib.clover_last_global_error()
    torch.cuda.synchronize()
    got = Y.cpu().numpy()
    assert np.all(got[:, N:] == -7.0)
    # products of N(0,1) and N(0,0.02): a sum of K terms is ~0.02 sqrt(K); planes of 16 mantissa bits are off by 2^-17 of it
    # (8e-6, a few sigma over all outputs: 4e-5 x 4), fp32 sums by less
    tol = (1e-5 if path == 0 else 4e-5) * np.sqrt(K) * 0.02 * 4
    err = np.abs(got[:, :N] - X.astype(np.float64) @ Wf.T).max()
    assert err <= tol, (err, tol)


# (M, N, K, RB, CB, row tiles, stages)
PLAIN = [
    (1, 26000, 128, 0, 4, 1, 2), (1, 34704, 128, 0, 6, 1, 2), (1, 16, 128, 1, 3, 1, 4), (17, 26000, 128, 1, 3.5, 1, 4),
    (17, 34704, 128, 1, 6, 1, 4), (33, 16, 128, 2, 3, 1, 4), (33, 26000, 128, 2, 3.5, 1, 4), (33, 34704, 128, 2, 6, 1, 4),
    (33, 52000, 128, 2, 8, 1, 4), (65, 16, 128, 3, 3, 1, 4), (97, 16, 128, 3, 3, 2, 4), (65, 26000, 128, 3, 4, 1, 4),
    (200, 8192, 128, 3, 4, 3, 4), (65, 34704, 128, 3, 6, 1, 4), (200, 10928, 128, 3, 6, 3, 4), (65, 52000, 128, 3, 7, 1, 4),
    (200, 17344, 128, 3, 7, 3, 4), (65, 58384, 128, 3, 8, 1, 4), (200, 19472, 128, 3, 8, 3, 4), (97, 26000, 128, 4, 4, 1, 4),
    (200, 16384, 128, 4, 4, 2, 4), (97, 34704, 128, 4, 6, 1, 4), (200, 21856, 128, 4, 6, 2, 4), (97, 52000, 128, 4, 7, 1, 4),
    (200, 26000, 128, 4, 7, 2, 4), (97, 58384, 128, 4, 8, 1, 4), (200, 29184, 128, 4, 8, 2, 4), (129, 29184, 128, 5, 4, 1, 4),
    (129, 34704, 128, 5, 6, 1, 4), (129, 52000, 128, 5, 7, 1, 4), (129, 58384, 128, 5, 8, 1, 4),
    (15, 26000, 640, 0, 4, 1, 10), (15, 34704, 640, 0, 6, 1, 10), (15, 16, 640, 1, 3, 1, 20), (15, 12992, 640, 1, 3.5, 1, 10),
    (15, 17344, 640, 1, 6, 1, 10), (50, 16, 640, 2, 3, 1, 20), (50, 12992, 640, 2, 3.5, 1, 10), (50, 34704, 640, 2, 6, 1, 20),
    (50, 52000, 640, 2, 8, 1, 20), (95, 16, 640, 3, 3, 1, 20), (127, 16, 640, 3, 3, 2, 20), (95, 26000, 640, 3, 4, 1, 20),
    (250, 8192, 640, 3, 4, 3, 20), (95, 34704, 640, 3, 6, 1, 20), (250, 10928, 640, 3, 6, 3, 20),
    (95, 52000, 640, 3, 7, 1, 20), (250, 17344, 640, 3, 7, 3, 20), (95, 58384, 640, 3, 8, 1, 20),
    (250, 19472, 640, 3, 8, 3, 20), (127, 26000, 640, 4, 4, 1, 20), (250, 16384, 640, 4, 4, 2, 20),
    (127, 34704, 640, 4, 6, 1, 20), (250, 21856, 640, 4, 6, 2, 20), (127, 52000, 640, 4, 7, 1, 20),
    (250, 26000, 640, 4, 7, 2, 20), (127, 58384, 640, 4, 8, 1, 20), (250, 29184, 640, 4, 8, 2, 20),
    (159, 29184, 640, 5, 4, 1, 20), (159, 34704, 640, 5, 6, 1, 20), (159, 52000, 640, 5, 7, 1, 20),
    (159, 58384, 640, 5, 8, 1, 20), (1, 16, 2176, 1, 3, 1, 17), (1, 6496, 2176, 1, 3.5, 1, 17), (1, 8672, 1920, 1, 6, 1, 15),
    (33, 16, 2176, 2, 3, 1, 17), (33, 6496, 1920, 2, 3.5, 1, 15), (33, 8672, 2176, 2, 6, 1, 17), (65, 16, 2176, 3, 3, 1, 17),
    (65, 6496, 2176, 3, 4, 1, 17), (65, 8672, 2176, 3, 6, 1, 17),
    # eight blocks for up to 64 rows: few and many stages, several ranges of K with odd and even stage counts
    (17, 28704, 128, 1, 4, 1, 4), (32, 28704, 640, 1, 4, 1, 20), (33, 28704, 128, 2, 4, 1, 4), (64, 29008, 640, 2, 4, 1, 20),
    (15, 14368, 640, 1, 4, 1, 10), (31, 14368, 640, 1, 4, 1, 10), (50, 14352, 2176, 2, 4, 1, 34), (1, 7712, 1920, 1, 4, 1, 15),
    (32, 7184, 2176, 1, 4, 1, 17), (33, 7200, 1920, 2, 4, 1, 15), (64, 8192, 2176, 2, 4, 1, 17), (9, 4096, 4096, 1, 4, 1, 16),
    (17, 4096, 4096, 1, 4, 1, 16), (64, 4096, 4096, 2, 4, 1, 16),
]
# (M, F, K, RB, CB, row tiles, stages)
SWIGLU = [
    (1, 12992, 128, 0, 4, 1, 2), (1, 17344, 128, 0, 6, 1, 2), (1, 32, 128, 1, 3, 1, 4), (17, 12992, 128, 1, 3.5, 1, 4),
    (17, 17344, 128, 1, 6, 1, 4), (33, 32, 128, 2, 3, 1, 4), (33, 12992, 128, 2, 3.5, 1, 4), (33, 17344, 128, 2, 6, 1, 4),
    (33, 27552, 128, 2, 8, 1, 4), (65, 32, 128, 3, 3, 1, 4), (97, 32, 128, 3, 3, 2, 4), (65, 12992, 128, 3, 4, 1, 4),
    (512, 2048, 128, 3, 4, 6, 4), (65, 17344, 128, 3, 6, 1, 4), (512, 2720, 128, 3, 6, 6, 4), (65, 27552, 128, 3, 7, 1, 4),
    (1000, 2432, 128, 3, 7, 11, 4), (65, 29184, 128, 3, 8, 1, 4), (700, 3648, 128, 3, 8, 8, 4), (97, 12992, 128, 4, 4, 1, 4),
    (512, 4096, 128, 4, 4, 4, 4), (97, 17344, 128, 4, 6, 1, 4), (640, 4864, 128, 4, 6, 5, 4), (97, 27552, 128, 4, 7, 1, 4),
    (400, 6880, 128, 4, 7, 4, 4), (97, 29184, 128, 4, 8, 1, 4), (1000, 3648, 128, 4, 8, 8, 4), (129, 14592, 128, 5, 4, 1, 4),
    (640, 4096, 128, 5, 4, 4, 4), (129, 17344, 128, 5, 6, 1, 4), (700, 4864, 128, 5, 6, 5, 4), (129, 27552, 128, 5, 7, 1, 4),
    (400, 8672, 128, 5, 7, 3, 4), (129, 29184, 128, 5, 8, 1, 4), (700, 5792, 128, 5, 8, 5, 4), (15, 12992, 640, 0, 4, 1, 10),
    (15, 17344, 640, 0, 6, 1, 10), (15, 32, 640, 1, 3, 1, 20), (31, 12992, 640, 1, 3.5, 1, 20), (31, 17344, 640, 1, 6, 1, 20),
    (50, 32, 640, 2, 3, 1, 20), (50, 12992, 640, 2, 3.5, 1, 20), (50, 17344, 640, 2, 6, 1, 20), (50, 27552, 640, 2, 8, 1, 20),
    (95, 32, 640, 3, 3, 1, 20), (127, 32, 640, 3, 3, 2, 20), (95, 12992, 640, 3, 4, 1, 20), (960, 1216, 640, 3, 4, 10, 20),
    (95, 17344, 640, 3, 6, 1, 20), (799, 1824, 640, 3, 6, 9, 20), (95, 27552, 640, 3, 7, 1, 20),
    (960, 2432, 640, 3, 7, 10, 20), (95, 29184, 640, 3, 8, 1, 20), (450, 5792, 640, 3, 8, 5, 20),
    (127, 12992, 640, 4, 4, 1, 20), (250, 8192, 640, 4, 4, 2, 20), (127, 17344, 640, 4, 6, 1, 20),
    (620, 4864, 640, 4, 6, 5, 20), (127, 27552, 640, 4, 7, 1, 20), (799, 3648, 640, 4, 7, 7, 20),
    (127, 29184, 640, 4, 8, 1, 20), (960, 4096, 640, 4, 8, 8, 20), (159, 14592, 640, 5, 4, 1, 20),
    (620, 4096, 640, 5, 4, 4, 20), (159, 17344, 640, 5, 6, 1, 20), (960, 3648, 640, 5, 6, 6, 20),
    (159, 27552, 640, 5, 7, 1, 20), (799, 5152, 640, 5, 7, 5, 20), (159, 29184, 640, 5, 8, 1, 20),
    (960, 4864, 640, 5, 8, 6, 20), (17, 14368, 128, 1, 4, 1, 4), (31, 16384, 640, 1, 4, 1, 20), (33, 14368, 128, 2, 4, 1, 4),
    (50, 16352, 640, 2, 4, 1, 20),
]


def _form(lib, epi, M, N, K):
    f, columns = (C.c_int32 * 5)(), C.c_int32()
    assert lib.clover_op_gemm_form(epi, M, N, K, 1 if epi else 0, f) == 0, lib.clover_last_global_error()
    assert lib.clover_op_gemm_tile_columns(epi, M, N, K, 1 if epi else 0, C.byref(columns)) == 0
    return f[0], columns.value / 32, f[2], f[4]


def _operands(torch, M, N, K, seed, n):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn(M, K, generator=gen, device="cuda")
    return X, [(torch.randn(N, K, generator=gen, device="cuda") * 0.02).bfloat16() for _ in range(n)]


def _ptr(t):
    return C.c_void_p(t.data_ptr())


@pytest.mark.parametrize("M,N,K,RB,CB,row_tiles,stages", PLAIN)
def test_plain_forms(M, N, K, RB, CB, row_tiles, stages):
    import torch
    print(f"gemm form RB={RB} CB={CB} M={M} N={N} K={K}", flush=True)
    lib = clover.load_library()
    assert _form(lib, 0, M, N, K) == (RB, CB, row_tiles, stages)
    X, (W,) = _operands(torch, M, N, K, M + N + K, 1)
    Y = torch.full((M, N), -7.0, device="cuda")
    nb = lib.clover_op_gemm_scratch_bytes(M, N, K)
    scratch = torch.full((nb,), 255, dtype=torch.uint8, device="cuda")   # (NaNs, as above)
    rc = lib.clover_op_gemm(7, 1, _ptr(X), _ptr(W), _ptr(Y), N, M, N, K, _ptr(scratch), nb,
                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lib.clover_last_global_error()
    tol = 4e-5 * np.sqrt(K) * 0.02 * 4                                   # (as above)
    err = (Y.double() - X.double() @ W.double().T).abs().max().item()
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("M,F,K,RB,CB,row_tiles,stages", SWIGLU)
def test_swiglu_forms(M, F, K, RB, CB, row_tiles, stages):
    import torch
    print(f"swiglu form RB={RB} CB={CB} M={M} F={F} K={K}", flush=True)
    lib = clover.load_library()
    assert _form(lib, 1, M, F, K) == (RB, CB, row_tiles, stages)
    X, (Wg, Wu) = _operands(torch, M, F, K, M + F + K, 2)
    mb = (M + 15) // 16
    planes = torch.full((F // 32, mb, 2, 16, 4, 8), -1, dtype=torch.int16, device="cuda")   # [step][row block][hi, lo][row][piece][column]
    nb = lib.clover_op_swiglu_scratch_bytes(M, F, K)
    scratch = torch.full((nb,), 255, dtype=torch.uint8, device="cuda")
    rc = lib.clover_op_swiglu(_ptr(X), _ptr(Wg), _ptr(Wu), _ptr(planes), M, F, K, _ptr(scratch), nb,
                              C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lib.clover_last_global_error()
    where = torch.tensor([[c ^ (-(r // 4) & 3) for c in range(4)] for r in range(16)], device="cuda")   # of piece c in row r
    bits = planes.gather(4, where[None, None, None, :, :, None].expand(planes.shape))
    rows = bits.permute(2, 1, 3, 0, 4, 5).reshape(2, mb * 16, F)                            # [hi, lo][row][column]
    assert bool((rows[:, M:] == -1).all())                                                  # rows past M stay as they were
    got = rows[:, :M].contiguous().view(torch.bfloat16).double().sum(0)
    g, u = X.double() @ Wg.double().T, X.double() @ Wu.double().T
    s = g * torch.sigmoid(g)
    # a product's error (the bound above) through the two factors (silu' <= 1.1), the planes' 16 mantissa bits
    tol = 4e-5 * np.sqrt(K) * 0.02 * 4 * (1.1 * u.abs() + s.abs()) + 2.0 ** -16 * (s * u).abs() + 1e-9
    bad = (got - s * u).abs() - tol
    assert bad.max().item() <= 0.0, (bad.max().item(), (bad > 0).nonzero()[:4].tolist())


@pytest.mark.parametrize("path,K", [(7, 640), (0, 260)])
def test_operands_off_the_16_byte_grid(path, K):
    """X may start on any 4 bytes and the rows of Y on any: the few-output kernel steps back to the tiles, the planes' reader
    takes it as it is"""
    import torch
    lib = clover.load_library()
    M, N = 33, 48
    X, (W,) = _operands(torch, M, N, K, K, 1)
    Xo = torch.empty(M * K + 1, device="cuda")[1:]
    Xo.copy_(X.flatten())
    Y = torch.full((M, N + 1), -7.0, device="cuda")
    nb = lib.clover_op_gemm_scratch_bytes(M, N, K)
    scratch = torch.full((nb,), 255, dtype=torch.uint8, device="cuda")
    rc = lib.clover_op_gemm(path, 1, _ptr(Xo), _ptr(W), _ptr(Y), N + 1, M, N, K, _ptr(scratch), nb,
                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lib.clover_last_global_error()
    assert (Y[:, :N].double() - X.double() @ W.double().T).abs().max().item() <= 4e-5 * np.sqrt(K) * 0.02 * 4
    assert bool((Y[:, N:] == -7.0).all())
