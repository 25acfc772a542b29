"""The 256-row tiles of the GEMM: the SwiGLU projection by itself, the plain product as the LM head of a verify pass
against the fp32-ALU kernels."""
import ctypes as C

import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth
from tests import test_gemm_tiles as tiles

pytestmark = pytest.mark.gpu

# (M, F, K, CB, row tiles, stages): a last row tile of 134, 74, 216, 11 and 153 rows, an odd stage count
SWIGLU = [(646, 6944, 4224, 6, 3, 132), (842, 6144, 1408, 6, 4, 44), (984, 6784, 1408, 7, 4, 44),
          (779, 8128, 1408, 8, 4, 44), (921, 7648, 1024, 8, 4, 32)]


@pytest.mark.parametrize("M,F,K,CB,row_tiles,stages", SWIGLU)
def test_swiglu_256_row_tiles(M, F, K, CB, row_tiles, stages):
    tiles.test_swiglu_forms(M, F, K, 8, CB, row_tiles, stages)


# (sequences, rows of the last one, vocabulary, CB): 512, 770 and 1024 rows
@pytest.mark.parametrize("batch,nodes,vocab,CB", [(4, 128, 16400, 6), (7, 2, 14352, 8), (8, 128, 12304, 7)])
def test_lm_head_256_row_tiles(batch, nodes, vocab, CB):
    import torch
    R = 128
    shape = synth.scaled(synth.CONFIGS[3], name="many-rows", n_layers=1, hidden=1024, n_q_heads=8, n_kv_heads=2, ffn=1536,
                         vocab=vocab, seed=5)
    M = (batch - 1) * R + nodes
    lib = clover.load_library()
    form = (C.c_int32 * 5)()
    assert lib.clover_op_gemm_form(0, M, vocab, 1024, 1, form) == 0 and tuple(form[:2]) == (8, CB), tuple(form)
    dev_w = clover.upload_weights(synth.WeightStore(shape))
    parent, rank = np.arange(-1, nodes - 1, dtype=np.int32), np.zeros(nodes, np.int32)
    tok = torch.randint(0, vocab, (batch, R), generator=torch.Generator().manual_seed(3)).int()
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, parent, rank, batch, 256, R, flags=flags)
        assert (g.path_info() & 1 == 1) == (flags == 0)
        g.tree_tokens.copy_(tok)
        g.logits.fill_(float("nan"))
        g.verify_tree(batch)
        torch.cuda.synchronize()
        out.append(g.logits[:, :nodes].double())
    # logits of N(0, 0.02) weights on normalised rows: 2^-17 of 0.02 sqrt(1024) per product (the bound of test_gemm_tiles,
    # 1e-4), a few times that for the layer in front
    err = (out[0] - out[1]).abs().max().item()
    assert err <= 5e-4, err
