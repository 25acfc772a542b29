"""The MFMA attention over sequences of unequal lengths, each with its own number of key ranges: lengths around a tile, one range
beside many, more sequences than the table of ranges holds, trees and interval labels, host bounds that lie above the
lengths on the device.  Reference: the fp32-ALU kernels on the same caches."""
import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
# (query heads per KV head, nodes, cached keys per sequence, interval labels, accept calls in front: each raises the host's bound)
CASES = [(4, 33, (0, 31, 700, 32, 2111, 64, 1), 0, 0), (4, 1, (5, 1500, 90), 0, 3), (4, 32, (1800, 256, 31, 900), 0, 2),
         (1, 65, (700, 12, 333), 1, 0), (2, 40, (64, 1000), 0, 1), (8, 17, (33, 640, 100, 2000), 0, 0),
         (4, 3, tuple(40 + (b * 37) % 300 for b in range(270)), 0, 0)]


@pytest.mark.parametrize("group,nodes,keys,interval,accepts", CASES)
def test_ragged_attention(group, nodes, keys, interval, accepts):
    import torch
    shape = synth.scaled(synth.CONFIGS[3], name="attn-ragged", n_layers=1, hidden=512, n_q_heads=8, n_kv_heads=8 // group, ffn=512,
                         vocab=4096, seed=17)
    dev_w = clover.upload_weights(synth.WeightStore(shape))
    rng = np.random.default_rng(nodes)
    parent = np.array([-1] + sorted(int(rng.integers(max(0, u // 3 - 2), u)) for u in range(1, nodes)), np.int32)
    rank = np.zeros(nodes, np.int32)
    for u in range(1, nodes):
        rank[u] = sum(parent[v] == parent[u] for v in range(1, u))
    batch, longest = len(keys), max(keys)
    K = rng.standard_normal((longest, shape.n_kv_heads, 128)).astype(np.float32)
    V = rng.standard_normal((longest, shape.n_kv_heads, 128)).astype(np.float32)
    max_seq = (longest + nodes * (accepts + 2) + 63) // 32 * 32
    tok = torch.randint(0, shape.vocab, (batch, nodes), generator=torch.Generator().manual_seed(1)).int()
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, parent, rank, batch, max_seq, nodes, flags=flags | (clover.FLAG_INTERVAL_MASK if interval else 0))
        for b in range(batch):
            if keys[b]:
                g.write_kv(0, 0, b, 0, K[:keys[b]], V[:keys[b]])
        g.set_seq_len(list(keys), [max(k - 1, 0) for k in keys])
        g.tree_tokens.copy_(tok)
        # (crafted logits accept the root alone: one key more per call, while the host must allow for the tree's depth)
        for _ in range(accepts):
            g.verify_tree(batch)
            g.logits.zero_()
            g.logits[:, :, 4095] = 1.0
            g.tree_tokens.clamp_(max=4094)
            g.accept_and_compact(batch)
        g.hidden.fill_(float("nan"))
        g.verify_tree(batch)
        torch.cuda.synchronize()
        out.append(g.hidden.double().cpu())
        del g
    # K, V, queries and probabilities carry 16 mantissa bits on one side (2^-17 each way); scores of N(0,1) keys against the
    # queries of this layer stay below 10, so a probability moves by 10 x 2^-16 and the attention's output (|V| below 5) by 1.5e-3,
    # 0.02 sqrt(1024) of it behind Wo and about as much again behind the FFN
    err = (out[0] - out[1]).abs().max().item()
    assert err <= 2e-3, err
