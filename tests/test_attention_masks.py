"""Who sees whom in the attention, where it shows: queries scaled so that soft-max weights are uneven, caches short enough that
the new rows carry the result, every form of the MFMA kernel (query heads per KV head, nodes per workgroup) around the 32, 64 and
128 nodes of a workgroup, bit sets and interval labels, and the chains of a prompt row by row.  Both routes are compared with the
oracle; on the CPU the oracle itself, with mistakes planted in its mask, shows that the bounds would see them."""
from functools import lru_cache

import numpy as np
import pytest

from oracle import clover2_oracle as O
from paper_2408_00264_amd import clover, synth

Q_HEADS = 8
# bound on a hidden row / on K and V of the second layer.  Scores reach 10 and operands carry 16 mantissa bits: 10 x 2^-16 of a
# probability, so 2e-4 of values of up to 1 in the attention's output, 0.02 sqrt(1024) = 0.64 of that behind Wo; the second
# layer's K is the normalised row (1 / 0.3) times 0.02 sqrt(512) = 0.45
BOUND = 3e-4

# (query heads per KV head, nodes, cached keys, interval labels): one split and several, tiles that end with the tree and not
TREES = [(1, 2, 0, 0), (1, 32, 5, 1), (1, 33, 31, 0), (1, 64, 40, 1), (1, 65, 0, 0), (1, 128, 33, 0), (1, 160, 20, 1), (2, 17, 3, 0),
         (2, 32, 32, 1), (2, 63, 1, 0), (2, 100, 70, 0), (2, 128, 0, 1), (4, 16, 31, 0), (4, 33, 0, 1), (4, 64, 64, 0), (4, 97, 2, 0),
         (4, 128, 90, 1), (8, 15, 40, 0), (8, 33, 33, 1), (8, 70, 0, 0), (8, 128, 7, 0), (3, 66, 9, 0)]
# (query heads per KV head, lengths of two prompts, one behind the other)
CHAINS = [(1, (20, 70)), (1, (129, 40)), (1, (300, 65)), (2, (31, 64)), (2, (140, 33)), (4, (33, 95)), (4, (257, 31)), (8, (40, 100)),
          (8, (160, 17)), (3, (66, 63))]


@lru_cache(maxsize=None)
def _model(group, layers):
    heads = 9 if group == 3 else Q_HEADS
    shape = synth.scaled(synth.CONFIGS[3], name="attn-masks", n_layers=layers, hidden=512, n_q_heads=heads, n_kv_heads=heads // group,
                         ffn=512, vocab=512, seed=37, ad_heads=8)
    plain = synth.WeightStore(shape)
    # (a power of two: the scaled weights are still bf16)
    over = {n: plain.get_f32(n) * np.float32(16.0) for n in plain.names() if n.endswith("wq") and n.startswith("layers")}
    return shape, synth.WeightStore(shape, overrides=over)


def _tree(nodes):
    rng = np.random.default_rng(nodes)
    parent = np.array([-1] + sorted(int(rng.integers(max(0, u // 3 - 2), u)) for u in range(1, nodes)), np.int32)
    rank = np.zeros(nodes, np.int32)
    for u in range(1, nodes):
        rank[u] = sum(parent[v] == parent[u] for v in range(1, u))
    return parent, rank


def _cached(shape, keys):
    rng = np.random.default_rng(keys)
    return [(0.45 * rng.standard_normal((keys, shape.n_kv_heads, 128))).astype(np.float32) for _ in range(2)]


def _oracle(shape, store, max_seq):
    cfg = O.OracleConfig.from_shape(shape, max_seq)
    return cfg, O.Weights(store.get_f32), O.SeqState(cfg)


def _tree_rows(case, vis=None):
    """hidden rows of the oracle, with the tree's own mask or another"""
    group, nodes, keys, _ = case
    shape, store = _model(group, 1)
    cfg, W, seq = _oracle(shape, store, keys + nodes)
    K, V = _cached(shape, keys)
    seq.kv.k[0, :keys], seq.kv.v[0, :keys] = K, V
    parent, _ = _tree(nodes)
    tok = np.random.default_rng(1).integers(0, shape.vocab, nodes)
    x = W("embed")[tok].astype(np.float64)
    return tok, O.decoder_layer(W, "layers.0.", cfg, x, seq.kv, 0, keys, keys + O.tree_depths(parent), keys + np.arange(nodes),
                                O.ancestor_matrix(parent) if vis is None else vis)


@pytest.mark.parametrize("case", TREES, ids=str)
def test_bound_sees_a_wrong_tree_mask(case):
    nodes, keys = case[1], case[2]
    true = O.ancestor_matrix(_tree(nodes)[0])
    rows = _tree_rows(case)[1]
    moved = lambda vis: np.abs(_tree_rows(case, vis)[1] - rows).max(axis=1)
    own = np.eye(nodes, dtype=bool)
    for wrong in (np.ones_like(true), own):          # all visible; a node alone: seen in every block of 16 nodes
        d = moved(wrong)
        for b in range(0, nodes, 16):
            assert d[b:b + 16].max() > 10 * BOUND, (b, d[b:b + 16].max())
    shifted = np.roll(true, 1, axis=1) | own          # the neighbour's column
    lost = true & (own | (np.arange(nodes)[None, :] % 64 != 0))     # the first bit of a word
    masks = [shifted, lost] + [true & (own | (np.arange(nodes)[None, :] // 64 != w)) for w in range((nodes + 63) // 64)]
    for wrong in masks:
        if (wrong != true).any():
            assert moved(wrong).max() > 10 * BOUND


@pytest.mark.gpu
@pytest.mark.parametrize("case", TREES, ids=str)
def test_tree_masks(case):
    import torch
    group, nodes, keys, interval = case
    shape, store = _model(group, 1)
    tok, want = _tree_rows(case)
    dev_w = clover.upload_weights(store)
    K, V = _cached(shape, keys)
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, *_tree(nodes), 1, (keys + nodes + 31) // 32 * 32, nodes,
                          flags=flags | (clover.FLAG_INTERVAL_MASK if interval else 0))
        assert g.path_info() == (0 if flags else 1 if group == 3 else 3)
        if keys:
            g.write_kv(0, 0, 0, 0, K, V)
        g.set_seq_len([keys], [0])
        g.tree_tokens.copy_(torch.from_numpy(tok.astype(np.int32))[None])
        g.hidden.fill_(float("nan"))
        g.verify_tree(1)
        torch.cuda.synchronize()
        err = np.abs(g.hidden[0].double().cpu().numpy() - want).max()
        print(f"{case} flags {flags}: {err:.1e}", flush=True)
        assert err <= BOUND, err
        g.close()


def _chain_rows(case, wrong=None):
    """K and V of the oracle's second layer behind both prompts; wrong(row, keys seen): another mask for the first layer"""
    group, lengths = case
    shape, store = _model(group, 2)
    cfg, W, seq = _oracle(shape, store, sum(lengths))
    toks, L = [], 0
    for n in lengths:
        tok = np.random.default_rng(n).integers(0, shape.vocab, n)
        toks.append(tok)
        pos, causal = L + np.arange(n), np.tril(np.ones((n, n), dtype=bool))
        vis = causal if wrong is None else wrong(causal.copy())
        x = W("embed")[tok].astype(np.float64)
        for li in range(2):
            x = O.decoder_layer(W, f"layers.{li}.", cfg, x, seq.kv, li, L, pos, pos, vis if li == 0 else causal)
        L += n
    return toks, seq.kv.k[1], seq.kv.v[1]


def _without_own(v):
    i = np.arange(1, len(v))
    v[i, i] = False
    return v


def _with_next(v):
    i = np.arange(len(v) - 1)
    v[i, i + 1] = True
    return v


def _without_last_tile(size):
    def wrong(v):                                    # the rows of a group of `size` lose the group's last 32 keys but their own
        n = len(v)
        for i in range(n):
            end = min(n, i // size * size + size)
            v[i, (end - 1) // 32 * 32:i] = False
        return v
    return wrong


@pytest.mark.parametrize("case", CHAINS, ids=str)
def test_bound_sees_a_wrong_causal_mask(case):
    _, k, v = _chain_rows(case)
    for wrong in (_without_own, _with_next, _without_last_tile(32), _without_last_tile(64), _without_last_tile(128)):
        _, k2, v2 = _chain_rows(case, wrong)
        d = np.maximum(np.abs(k2 - k), np.abs(v2 - v)).max(axis=(1, 2))
        changed, L = np.zeros(len(d), dtype=bool), 0
        for n in case[1]:
            causal = np.tril(np.ones((n, n), dtype=bool))
            changed[L:L + n] = (wrong(causal.copy()) != causal).any(axis=1)
            L += n
        for b in range(0, len(d), 16):               # in every 16 rows that the mistake touches, a prompt's last among them
            if changed[b:b + 16].any():
                assert d[b:b + 16].max() > 3 * BOUND, (b, d[b:b + 16].max())
        assert np.mean(d[changed] > BOUND) > 0.9


@pytest.mark.gpu
@pytest.mark.parametrize("case", CHAINS, ids=str)
def test_prompts_row_by_row(case):
    import torch
    group, lengths = case
    shape, store = _model(group, 2)
    toks, k, v = _chain_rows(case)
    dev_w = clover.upload_weights(store)
    total = sum(lengths)
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, np.asarray([-1], np.int32), np.asarray([0], np.int32), 1, (total + 31) // 32 * 32, 1,
                          flags=flags, prefill_rows=256)
        for t in toks:
            g.prefill_prompt(0, torch.from_numpy(t.astype(np.int32)).cuda())
        got = g.read_kv(0, 1, 0, 0, total)
        err = max(np.abs(got[0] - k).max(), np.abs(got[1] - v).max())
        print(f"{case} flags {flags}: {err:.1e}", flush=True)
        assert err <= BOUND, err
        g.close()
