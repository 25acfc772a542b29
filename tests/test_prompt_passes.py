"""The passes of the prefill call: as many rows as the memory of a step's buffers holds, whatever prefill_rows says, the same
state behind them, and nothing of a step in flight disturbed."""
import ctypes as C

import numpy as np
import pytest
import torch   # (in front of the library: a process has one HIP runtime, torch's own)

from paper_2408_00264_amd import clover, synth

MINI = synth.scaled(synth.CONFIGS[3], name="mini-passes", n_layers=2, hidden=512, n_q_heads=4, n_kv_heads=2, ffn=1536,
                    vocab=8192, tree_k=(4, 3, 2, 2), tree_nodes=24, seed=19)


def _bytes(shape, batch, max_seq, nodes, flags, prefill_rows):
    n = C.c_size_t()
    cfg = clover.make_config(shape, batch, max_seq, nodes, flags, prefill_rows)
    assert clover.load_library().clover_workspace_bytes(C.byref(cfg), C.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("shape,batch,max_seq,nodes,flags", [
    (synth.CONFIGS[1], 1, 256, 16, 0), (synth.CONFIGS[2], 1, 1280, 64, 0), (synth.CONFIGS[3], 1, 8448, 64, 0),
    (synth.CONFIGS[3], 1, 1280, 64, clover.FLAG_GENERIC), (synth.CONFIGS[4], 4, 2560, 32, 0), (MINI, 2, 768, 24, 0)])
def test_workspace_grows_by_the_row(shape, batch, max_seq, nodes, flags):
    """no value of prefill_rows costs more than its rows: steps of at most twice the one before (the row blocks of the planes)"""
    size = [_bytes(shape, batch, max_seq, nodes, flags, r) for r in (0, 127, 200, 224, 240, 254, 255, 256)]
    assert size == sorted(size)
    assert size[7] - size[6] <= 2 * (size[6] - size[5]), size
    assert _bytes(shape, batch, max_seq, 1, flags, 256) <= size[7]


def _tree(shape):
    return synth.make_tree(shape.tree_k, shape.tree_nodes)


def _prompt(shape, n, seed):
    return torch.randint(0, shape.vocab, (n,), generator=torch.Generator().manual_seed(seed)).int().cuda()


def _prefill(shape, dev_w, n, max_seq, prefill_rows, flags=0, shuffled=False):
    """(passes, K and V of the last layer, those of the Augmenting Block, logits, hidden) of one prompt"""
    g = clover.Clover(shape, dev_w, *_tree(shape), 1, max_seq, shape.tree_nodes, flags=flags, prefill_rows=prefill_rows)
    if shuffled:
        g.set_page_table(np.random.default_rng(n).permutation(max_seq // 32).astype(np.int32))
    g.profile_enable(True)
    g.prefill_prompt(0, _prompt(shape, n, n))
    torch.cuda.synchronize()
    embeds = g.profile_collect()["embed"][1]       # one for the target and one for the draft side of every pass
    out = [*g.read_kv(0, shape.n_layers - 1, 0, 0, n), *g.read_kv(1, 0, 0, 0, n - 1), g.logits[0, 0].cpu().numpy(),
           g.hid_acc[0, 0].cpu().numpy()]
    assert g.seq_len()[0] == n
    g.close()
    return (embeds + 1) // 2, out


# (model, prompt, prefill_rows of the two sides, flags; the first side's pages are shuffled): around whole passes, one row left, the fp32-ALU route and
# fp32; LLaMA3-8B widths: passes of 2048 rows against 512-row ones
CASES = [(MINI, 600, 0, 256, 0), (MINI, 256, 0, 255, 0), (MINI, 257, 0, 256, 0), (MINI, 513, 1, 64, 0),
         (MINI, 600, 0, 200, clover.FLAG_GENERIC), (synth.scaled(synth.CONFIGS[1], seed=20), 500, 0, 256, 0),
         (synth.scaled(synth.CONFIGS[3], name="wide-passes", n_layers=2, seed=21), 4173, 256, 0, 0),
         (synth.scaled(MINI, name="plain-gate", ad_heads=256, seed=22), 600, 0, 256, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[f"{c[0].name}-{c[1]}-{c[2]}-{c[4]}" for c in CASES])
def test_state_does_not_depend_on_the_passes(case):
    shape, n, rows_a, rows_b, flags = case
    dev_w = clover.upload_weights(synth.WeightStore(shape))
    max_seq = (n + 95) // 32 * 32
    p_a, a = _prefill(shape, dev_w, n, max_seq, rows_a, flags, shuffled=True)
    p_b, b = _prefill(shape, dev_w, n, max_seq, rows_b, flags)
    print(f"{shape.name}: {n} tokens in {p_a} and {p_b} passes", flush=True)
    assert max(p_a, p_b) > 1 or n <= 256
    if n == 4173:
        assert (p_a, p_b) == (3, 9)                # 2048 + 2048 + 77 rows; 512 each
    # the bounds of every model test: K/V rows 2e-3 (a lost low plane shows as 1e-2), hidden 1e-2, logits 3e-2; fp32 1e-4
    tol = [2e-3] * 4 + [3e-2, 1e-2] if shape.bf16 else [1e-4] * 6
    for x, y, t in zip(a, b, tol):
        assert np.isfinite(x).all() and np.abs(x - y).max() <= t, np.abs(x - y).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dynamic", [False, True])
def test_prompt_of_another_sequence_between_the_calls_of_a_step(dynamic):
    """draft_tree, verify_tree and accept_and_compact of sequence 0 with a prompt of sequence 1 in front of each: the same
    tokens, logits and cache rows, bit by bit (one batch size, so the same launches)"""
    dev_w = clover.upload_weights(synth.WeightStore(MINI))
    got = []
    for between in (False, True):
        g = clover.Clover(MINI, dev_w, *_tree(MINI), 2, 512, 24)
        g.prefill_prompt(0, _prompt(MINI, 300, 1))
        g.m.zero_()
        g.m[0] = 1
        if dynamic:
            g.set_dynamic_tree(24, 4, 4)

        def prompt():
            if between:
                keep = g.logits.clone(), g.hid_acc.clone(), g.next_tok.clone()
                g.prefill_prompt(1, _prompt(MINI, 80, 2))
                for t, k in zip((g.logits, g.hid_acc, g.next_tok), keep):
                    t.copy_(k)                     # (the binding hands the prompt's outputs over in the step's buffers)
        out = []
        for _ in range(2):
            prompt()
            g.draft_tree(1)
            out.append(g.tree_tokens[0].clone())
            prompt()
            g.verify_tree(1)
            out += [g.logits[0].clone(), g.hidden[0].clone()]
            prompt()
            g.accept_and_compact(1)
            out += [g.m[0].clone(), g.acc_idx[0].clone(), g.new_tokens[0].clone()]
        n = int(g.seq_len()[0])
        out += [torch.from_numpy(t) for t in g.read_kv(0, 1, 0, 0, n)]
        got.append(out)
        g.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)
