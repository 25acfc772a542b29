"""The MFMA tree attention against the fp32-ALU kernels on the same caches: every form (query heads per KV head, nodes per
workgroup), trees and interval labels around the 32, 64 and 128 nodes of a workgroup, caches around a tile, over 64 tiles
unsplit and over several splits, and scores that grow along the cache so that the reference of the soft-max moves.  (With
these scores the new rows hardly count: test_attention_masks.py has the masks.)"""
import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
Q_HEADS = 8
# (query heads per KV head, nodes, cached keys, batch, interval labels)
CASES = [(1, 1, 31, 1, 0), (1, 33, 64, 2, 0), (1, 65, 97, 1, 1), (1, 128, 700, 8, 0), (2, 32, 95, 1, 1), (2, 65, 33, 2, 0),
         (4, 5, 0, 1, 0), (4, 32, 4100, 64, 0), (4, 33, 2111, 1, 0), (4, 96, 500, 1, 1), (8, 31, 160, 1, 0), (8, 70, 333, 2, 0)]


def _weights_and_shape(group):
    shape = synth.scaled(synth.CONFIGS[3], name="attn-forms", n_layers=1, hidden=512, n_q_heads=Q_HEADS, n_kv_heads=Q_HEADS // group,
                         ffn=512, vocab=4096, seed=17)
    return shape, clover.upload_weights(synth.WeightStore(shape))


@pytest.mark.parametrize("group,nodes,keys,batch,interval", CASES)
def test_attention_forms(group, nodes, keys, batch, interval):
    import torch
    shape, dev_w = _weights_and_shape(group)
    rng = np.random.default_rng(nodes + keys)
    parent = np.array([-1] + sorted(int(rng.integers(max(0, u // 3 - 2), u)) for u in range(1, nodes)), np.int32)
    rank = np.zeros(nodes, np.int32)
    for u in range(1, nodes):
        rank[u] = sum(parent[v] == parent[u] for v in range(1, u))
    n_kv = shape.n_kv_heads
    # keys whose scores grow along the cache (up to about 60), so that later tiles exceed the reference of the first ones
    K = [(rng.standard_normal((keys, n_kv, 128)) * (1.0 + 30.0 * np.arange(keys)[:, None, None] / max(keys, 1))).astype(np.float32)
         for _ in range(min(batch, 2))]
    V = [rng.standard_normal((keys, n_kv, 128)).astype(np.float32) for _ in K]
    max_seq = (keys + nodes + 63) // 32 * 32
    tok = torch.randint(0, shape.vocab, (batch, nodes), generator=torch.Generator().manual_seed(1)).int()
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        b_run = batch if flags == 0 else min(batch, 2)   # (sequences repeat with period 2)
        g = clover.Clover(shape, dev_w, parent, rank, b_run, max_seq, nodes, flags=flags | (clover.FLAG_INTERVAL_MASK if interval else 0))
        assert g.path_info() == (3 if flags == 0 else 0)
        for b in range(b_run if keys else 0):
            g.write_kv(0, 0, b, 0, K[b % len(K)], V[b % len(K)])
        g.set_seq_len([keys] * b_run, [max(keys - 1, 0)] * b_run)
        g.tree_tokens.copy_(torch.stack([tok[b % len(K)] for b in range(b_run)]))
        g.hidden.fill_(float("nan"))
        g.verify_tree(b_run)
        torch.cuda.synchronize()
        out.append(g.hidden.double().cpu())
        del g
    # both sides read the same K and V to 16 mantissa bits; the MFMA side's queries (16 bits) move a score of 60 by 60 x 2^-17 =
    # 5e-4 and a probability by that share: up to 2 x 5e-4 x |V| (4) on the attention's output, 0.02 sqrt(1024) = 0.64 of it
    # behind Wo, about as much again behind the FFN
    err = max((out[0][b] - out[1][b % len(out[1])]).abs().max().item() for b in range(batch))
    assert err <= 6e-3, err


@pytest.mark.parametrize("group,lengths", [(4, (33, 600)), (1, (129, 1100)), (2, (65, 64)), (8, (100, 300))])
def test_prompt_attention(group, lengths):
    """chains: whole prompts in one pass (every tile holds new rows), then a second prompt behind the first"""
    import torch
    shape, dev_w = _weights_and_shape(group)
    toks = [torch.randint(0, shape.vocab, (n,), generator=torch.Generator().manual_seed(n)).int().cuda() for n in lengths]
    out = []
    for flags, rows in ((0, 256), (clover.FLAG_GENERIC, 128)):
        g = clover.Clover(shape, dev_w, np.asarray([-1], np.int32), np.asarray([0], np.int32), 1, 1280, 1, flags=flags, prefill_rows=rows)
        got = []
        for t in toks:
            g.prefill_prompt(0, t)
            got += [g.logits[0, 0].double().cpu(), g.hid_acc[0, 0].double().cpu()]
        out.append(got)
        del g
    # activations of 16 mantissa bits through one layer: 1e-4 on the logits (the bound of test_gemm_tiles), four times that
    for a, b in zip(*out):
        assert (a - b).abs().max().item() <= 4e-4, (a - b).abs().max().item()
