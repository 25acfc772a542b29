"""What earlier calls left in the caches behind a sequence's last key, and in the query rows behind its last new row, must not
reach a result in any bit: the MFMA attention multiplies such rows along with the valid ones of their block."""
import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
GROUPS = [1, 2, 4, 8]          # query heads per KV head: every form of the kernel
CACHED = 300


def _context(group, nodes=16):
    shape = synth.scaled(synth.CONFIGS[3], name="attn-leftovers", n_layers=1, hidden=512, n_q_heads=8, n_kv_heads=8 // group, ffn=512,
                         vocab=4096, seed=23)
    parent = np.array([-1, 0, 0, 1, 3], np.int32)
    return clover.Clover(shape, clover.upload_weights(synth.WeightStore(shape)), parent, np.array([0, 0, 1, 0, 0], np.int32), 1, 512, nodes)


def _keys(g, n, seed, scale):
    rng = np.random.default_rng(seed)
    return [(rng.standard_normal((n, g.shape.n_kv_heads, 128)) * s).astype(np.float32) for s in (scale, 1.0)]


@pytest.mark.parametrize("group", GROUPS)
@pytest.mark.parametrize("rows", [1, 21, 70])
def test_prompt_behind_a_longer_sequence(group, rows):
    import torch
    out = []
    for scale in (0.0, 1000.0):    # keys that a longer sequence has left behind the prompt's last position
        g = _context(group)
        g.write_kv(0, 0, 0, 0, *_keys(g, CACHED, 1, 4.0))
        g.write_kv(0, 0, 0, CACHED + rows, *_keys(g, 512 - CACHED - rows, 2, scale))
        g.set_seq_len([CACHED], [0])
        g.prefill_prompt(0, torch.arange(1, rows + 1, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        out.append((g.logits[0, 0].cpu(), g.hid_acc[0, 0].cpu()))
    assert torch.isfinite(out[0][0]).all()
    for a, b in zip(*out):
        assert torch.equal(a, b), (a - b).abs().max().item()


@pytest.mark.parametrize("group", GROUPS)
@pytest.mark.parametrize("m", [1, 3, 15])
def test_draft_behind_a_longer_draft(group, m):
    import torch
    gen = torch.Generator().manual_seed(m)
    hid, tok = torch.randn(24, 1, 16, 512, generator=gen), torch.randint(0, 4096, (24, 1, 16), generator=gen).int()
    keys = None
    out = []
    for first in range(1, 24):     # the rows that an earlier draft has left behind this one's m
        if keys is None:
            g = _context(group)
            captured = g.capture_draft_logits()
            keys = _keys(g, CACHED, 3, 12.0)
        for i, n in ((first, 16), (0, m)):
            g.set_seq_len([0], [CACHED])
            g.write_kv(1, 0, 0, 0, *keys)
            g.hid_acc.copy_(hid[i])
            g.next_tok.copy_(tok[i])
            g.m.fill_(n)
            g.draft_tree(1)
        torch.cuda.synchronize()
        out.append(captured[:4].cpu())
    assert torch.isfinite(out[0]).all() and out[0].abs().max() > 0
    for o in out[1:]:
        assert torch.equal(out[0], o), (out[0] - o).abs().max().item()
