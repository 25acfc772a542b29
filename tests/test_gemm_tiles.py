"""The GEMM kernels at the edges of their tiles: every row class and column remainder of the MFMA kernel, and the
few-output fp32 kernel at one row, one column, K tails and the tile count where the larger tiles take over."""
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
