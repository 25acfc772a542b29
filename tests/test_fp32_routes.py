"""fp32-ALU products on either side of the rules that choose their launches: joint with the norm or by themselves, one to four
wavefronts over K.  The rows of a pass do not depend on each other, so many equal sequences must give what one gives."""
import ctypes as C

import numpy as np
import pytest
import torch   # (in front of the library: a process has one HIP runtime, torch's own)

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
SHAPE = synth.scaled(synth.CONFIGS[1], name="fp32-routes", n_layers=1, hidden=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=1540,
                     vocab=4096, seed=29)


def _verify(dev_w, batch, nodes):
    parent, rank = np.arange(-1, nodes - 1, dtype=np.int32), np.zeros(nodes, np.int32)
    g = clover.Clover(SHAPE, dev_w, parent, rank, batch, 128, nodes)
    tok = torch.randint(0, SHAPE.vocab, (1, nodes), generator=torch.Generator().manual_seed(3)).int()
    g.tree_tokens.copy_(tok.expand(batch, nodes))
    g.profile_enable(True)
    g.verify_tree(batch)
    torch.cuda.synchronize()
    n = {k: v[1] for k, v in g.profile_collect().items()}
    return g.logits.double(), g.hidden.double(), n


# (sequences, launches of: norm, QKV, gate+up, LM head)
@pytest.mark.parametrize("batch,want", [(1, (0, 1, 1, 1)), (2, (1, 1, 1, 1)), (6, (2, 1, 2, 1)), (21, (3, 3, 2, 1))])
def test_rows_do_not_depend_on_the_route(batch, want):
    dev_w = clover.upload_weights(synth.WeightStore(SHAPE))
    l1, h1, _ = _verify(dev_w, 1, 64)
    l, h, n = _verify(dev_w, batch, 64)
    assert tuple(n[k] for k in ("rmsnorm", "gemm_qkv", "gemm_gate_up", "gemm_lm_head")) == want, n
    # the same fp32 sums in another order: 4 eps sqrt(1024) of unit-size terms times 0.02, the layer's outputs of up to 1
    for b in range(batch):
        assert (l[b] - l1[0]).abs().max().item() <= 1e-5 and (h[b] - h1[0]).abs().max().item() <= 1e-5


# blocks of 16 x 4 outputs: 512 | 516, 1024 | 1028, each with a K that ends inside a wavefront's first, second and third part
@pytest.mark.parametrize("dtype", [clover.DTYPE_F32, clover.DTYPE_BF16])
@pytest.mark.parametrize("M,N,K", [(16, 2048, 1020), (16, 2064, 516), (16, 4096, 260), (16, 4112, 1284), (33, 1363, 772), (63, 1024, 1000)])
def test_product_over_shared_k(dtype, M, N, K):
    X, W, Y = _product(dtype, M, N, K)
    err = (Y.double() - X.double() @ W.double().T).abs().max().item()
    assert err <= 1e-5 * K ** 0.5 * 0.02 * 4, err   # (the bound of the fp32 GEMM tests)


def _product(dtype, M, N, K):
    lib = clover.load_library()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    X = torch.randn(M, K, generator=gen, device="cuda")
    W = torch.randn(N, K, generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16 if dtype == clover.DTYPE_BF16 else torch.float32)
    Y = torch.full((M, N), float("nan"), device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    p = lambda t: C.c_void_p(t.data_ptr())
    assert lib.clover_op_gemm(0, dtype, p(X), p(W), p(Y), N, M, N, K, p(Y), 0, C.c_void_p(st)) == 0
    return X, W, Y


# tiles of 64 x 64: 256, 752 | 768, at a K of 256 368 | 384: the longer passes of a prompt take the sums of a few rows
@pytest.mark.parametrize("M,N,K,same", [(256, 4096, 516, True), (1000, 3000, 260, True), (1010, 3060, 260, False), (1000, 1450, 256, True),
                                        (1024, 1536, 256, False)])
def test_products_up_to_three_tiles_a_compute_unit(M, N, K, same):
    X, W, Y = _product(clover.DTYPE_F32, M, N, K)
    err = (Y.double() - X.double() @ W.double().T).abs().max().item()
    assert err <= 1e-5 * K ** 0.5 * 0.02 * 4, err
    few = torch.empty(64, N, device="cuda")      # more than 1024 blocks too, so one wavefront to a block in both
    p = lambda t: C.c_void_p(t.data_ptr())
    assert clover.load_library().clover_op_gemm(0, clover.DTYPE_F32, p(X), p(W), p(few), N, 64, N, K, p(few), 0,
                                                C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert torch.equal(few, Y[:64]) == same
