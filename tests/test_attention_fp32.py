"""The attention over fp32 caches: lengths around a tile of 64 keys and around a page, last tiles that end with the cache, one, two and
four wavefronts to a row and head, some of them without a tile; trees by bit sets and by labels, prompt chains, both head sizes, groups
of heads, several sequences.  Reference: the oracle."""
import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
# (query heads, KV heads, head size, nodes, cached keys per sequence, max_seq, labels): up to 512 rows x heads are four wavefronts
# each, up to 1024 two
CASES = [(4, 2, 64, 1, (1,), 64, 0), (4, 2, 64, 1, (63,), 96, 0), (4, 4, 64, 3, (61,), 96, 1), (4, 1, 64, 17, (47,), 128, 0),
         (4, 2, 64, 16, (64, 33, 200), 288, 0), (4, 2, 64, 128, (300,), 512, 0), (4, 2, 64, 120, (65, 257), 512, 1),
         (8, 2, 64, 65, (129,), 256, 0), (8, 8, 64, 128, (70,), 256, 0), (9, 3, 64, 114, (31,), 160, 0),
         (2, 1, 128, 1, (95,), 128, 0), (2, 2, 128, 33, (64, 190), 288, 1), (4, 1, 128, 128, (100,), 256, 0), (8, 4, 128, 100, (33, 1), 192, 0)]


@pytest.mark.parametrize("n_q,n_kv,d,nodes,keys,max_seq,labels", CASES)
def test_steps(n_q, n_kv, d, nodes, keys, max_seq, labels):
    import torch
    assert torch.cuda.is_available()
    from tests.parity import Lockstep
    shape = synth.scaled(synth.CONFIGS[1], name="attn-fp32", n_layers=1, hidden=36 * n_q, ffn=132, vocab=512, n_q_heads=n_q, n_kv_heads=n_kv,
                         head_dim=d, batch=len(keys), tree_k=(8, 6, 4, 3), tree_nodes=nodes, draft_depths=4, seed=29)
    parent, rank = synth.tree_for(shape)
    ls = Lockstep(shape, parent, rank, batch=len(keys), max_seq=max_seq, flags=clover.FLAG_INTERVAL_MASK if labels else 0)
    print(f"attention fp32: {len(keys) * nodes * n_q} rows x heads, keys {keys}", flush=True)
    ls.seed_cache(list(keys), nodes)
    ls.step()
    assert ls.max_logit_err <= 1e-4, ls.max_logit_err   # (the fp32 bound of every model test)


@pytest.mark.parametrize("n_q,d,n", [(4, 64, 130), (4, 64, 257), (2, 128, 97)])
def test_prompts(n_q, d, n):
    """chains: a row's last tile is its own"""
    import torch
    assert torch.cuda.is_available()
    from tests.parity import Lockstep
    shape = synth.scaled(synth.CONFIGS[1], name="attn-fp32-chain", n_layers=2, hidden=64 * n_q, ffn=132, vocab=512, n_q_heads=n_q, n_kv_heads=2,
                         head_dim=d, tree_k=(3, 2), tree_nodes=7, draft_depths=2, seed=31)
    parent, rank = synth.tree_for(shape)
    ls = Lockstep(shape, parent, rank, max_seq=320, prefill_rows=100)
    ls.prefill_prompts([np.random.default_rng(n).integers(0, 512, size=n).astype(np.int32)], oracle_chunk=64)
    ls.step()
    assert ls.max_logit_err <= 1e-4, ls.max_logit_err


# three tiles of 64 keys and a part of a fourth, so that of four wavefronts each has one
NAN_TILES = {"first": slice(0, 64), "second": slice(64, 128), "second and third": slice(64, 192), "one key": slice(130, 131)}


def _poisoned(batch, keys, value, channel=None):
    """hidden rows of sequence 0 whose cached keys `keys` hold `value` (in one channel, the others zero), beside sequences that do not"""
    import torch
    assert torch.cuda.is_available()
    shape = synth.scaled(synth.CONFIGS[1], name="attn-fp32-nan", n_layers=1, hidden=128, ffn=132, vocab=512, n_q_heads=2, n_kv_heads=1, head_dim=64,
                         batch=batch, tree_k=(4, 3, 2), tree_nodes=16, draft_depths=3, seed=37)
    parent, rank = synth.tree_for(shape)
    g = clover.Clover(shape, clover.upload_weights(synth.WeightStore(shape)), parent, rank, batch, 256, 16)
    rng = np.random.default_rng(5)
    k, v = (rng.standard_normal((200, 1, 64)).astype(np.float32) for _ in range(2))
    for b in range(batch):
        kb = k.copy()
        if b == 0 and channel is None:
            kb[keys] = value
        elif b == 0:
            kb[keys] = 0.0
            kb[keys, :, channel] = value
        g.write_kv(0, 0, b, 0, kb, v)
    g.set_seq_len([200] * batch, [0] * batch)
    gen = torch.Generator().manual_seed(2)
    g.tree_tokens.copy_(torch.randint(0, 512, (16,), generator=gen).int().expand(batch, 16))
    g.verify_tree(batch)
    torch.cuda.synchronize()
    out = g.hidden.double().cpu()
    g.close()
    return out


@pytest.mark.parametrize("where", NAN_TILES)
def test_keys_that_are_no_number(where):
    """A row that sees one has no result, however many wavefronts share its tiles: 4, 2 and 1 at these batches (32 rows x heads each)."""
    import torch
    for batch in (1, 20, 35):
        out = _poisoned(batch, NAN_TILES[where], np.nan)
        assert torch.isnan(out[0]).all(), (where, batch, torch.isnan(out[0]).sum().item())
        assert torch.isfinite(out[1:]).all()


@pytest.mark.parametrize("where", NAN_TILES)
def test_scores_of_minus_infinity(where):
    """A key of infinite size: rows that point away from it in both heads leave it out, the others have no result; the same rows and the
    same values however many wavefronts share the tiles."""
    import torch
    outs = [_poisoned(batch, NAN_TILES[where], np.inf, channel=9)[0] for batch in (1, 20, 35)]
    whole = torch.isfinite(outs[0]).all(dim=-1)
    assert 0 < whole.sum() < len(whole), whole
    for o in outs[1:]:
        assert torch.equal(torch.isnan(o), torch.isnan(outs[0]))
        assert (o[whole] - outs[0][whole]).abs().max().item() <= 1e-4    # (the fp32 bound of every model test)
