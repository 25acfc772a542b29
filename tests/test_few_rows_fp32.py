"""fp32 models at the edges of the few-row kernels (norm, joint projections and SwiGLU in the GEMM; attention by 16-byte pieces):
widths that are no multiple of 64, 256 or 16, one row to more than one row block, a second wavefront of K with a tail."""
import numpy as np
import pytest

from paper_2408_00264_amd import synth

pytestmark = pytest.mark.gpu


# (hidden, ffn, vocabulary, query heads, KV heads, head dim, tree, prompt)
@pytest.mark.parametrize("H,F,V,nq,nkv,d,tree,n", [
    (260, 516, 1023, 4, 2, 64, ((4, 3, 2), 17), 40), (256, 1028, 2049, 2, 1, 128, ((1,), 1), 65),
    (1036, 132, 130, 4, 4, 64, ((4, 4, 2), 33), 64), (64, 44, 2048, 1, 1, 64, ((3, 2), 10), 1)])
def test_fp32_steps(H, F, V, nq, nkv, d, tree, n):
    import torch
    assert torch.cuda.is_available()
    from tests.parity import Lockstep
    k, nodes = tree
    shape = synth.scaled(synth.CONFIGS[1], name="few-rows-fp32", hidden=H, ffn=F, vocab=V, n_q_heads=nq, n_kv_heads=nkv, head_dim=d,
                         tree_k=k, tree_nodes=nodes, draft_depths=max(len(k), 1), seed=23)
    parent, rank = synth.tree_for(shape)
    ls = Lockstep(shape, parent, rank, max_seq=160, gain_jitter=0.1, prefill_rows=48)
    rng = np.random.default_rng(H)
    ls.prefill_prompts([rng.integers(0, V, size=n).astype(np.int32)], oracle_chunk=32)
    for _ in range(2):
        ls.step()
    assert ls.max_logit_err <= 1e-4, ls.max_logit_err   # (the fp32 bound of every model test)
