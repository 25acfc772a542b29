"""The QKV projection, its rotation and its way into the caches, in one launch or two: tiles over one and several ranges of K, whole and
partial row blocks and last tiles, sequences with unused rows between them, both head sizes, shuffled pages.  Reference: the
fp32-ALU kernels of the same model.  Which launches ran is asserted by the profile."""
import ctypes as C

import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

# (hidden, query heads, KV heads, head size, sequences, nodes, rows of a sequence, K ranges that the rule takes, launches)
CASES = [(4096, 32, 8, 128, 1, 1, 1, 8, 2), (4096, 32, 8, 128, 1, 16, 24, 8, 2), (4096, 32, 8, 128, 1, 17, 17, 8, 2), (4096, 32, 8, 128, 2, 30, 33, 4, 1),
         (4096, 32, 8, 128, 3, 32, 32, 4, 1), (4096, 32, 8, 128, 1, 120, 128, 4, 2), (4096, 32, 8, 128, 8, 32, 32, 4, 2),
         (1024, 8, 2, 128, 1, 5, 5, 4, 1), (1024, 8, 2, 128, 3, 50, 60, 4, 2), (640, 5, 5, 128, 2, 9, 40, 2, 2),
         (512, 32, 32, 128, 12, 50, 51, 1, 2), (2048, 16, 16, 128, 9, 60, 60, 1, 2),
         # few rows of two ranges; the widest tiles of up to 64 rows; tiles of 96 and 128, whose last row block is not whole
         (640, 5, 5, 128, 1, 9, 9, 2, 1), (4096, 32, 32, 128, 1, 8, 8, 4, 1), (5120, 40, 40, 128, 1, 49, 49, 4, 1), (4096, 32, 32, 128, 2, 41, 50, 4, 1),
         (2560, 20, 20, 128, 1, 83, 83, 4, 1), (2560, 20, 20, 128, 1, 118, 128, 4, 1), (3072, 24, 24, 128, 4, 27, 28, 3, 1),
         # short ranges; several row tiles with their ranges on several XCDs; more than 128 rows
         (1024, 8, 2, 128, 3, 30, 33, 4, 2), (3072, 24, 24, 128, 1, 160, 160, 3, 2), (2560, 20, 20, 128, 1, 133, 133, 4, 2)]


# (the library's own functions, by their C++ names)
def _ranges(M, N, K):
    return clover.load_library()._ZN3clv22tile_gemm_pick_k_partsEiii(M, N, K)


def _joins(M, N, K, ranges, mfma_attention):
    """whether one launch does it all, and its (row blocks / 2, column blocks, row tiles, ranges, stages)"""
    form = (C.c_int * 5)()
    f = clover.load_library()._ZN3clv19tile_gemm_qkv_joinsEiiiibPNS_8TileFormE
    f.restype, f.argtypes = C.c_bool, [C.c_int] * 4 + [C.c_bool, C.c_void_p]
    return f(M, N, K, ranges, mfma_attention, form), list(form)


def _model(H, n_q, n_kv, d, batch, nodes, R):
    """(shape, weights, parents, ranks, cached rows, slots, page table, tokens) of a model of one layer"""
    import torch
    assert torch.cuda.is_available()
    M = (batch - 1) * R + nodes
    print(f"qkv M={M} N={(n_q + 2 * n_kv) * d} K={H}", flush=True)
    shape = synth.scaled(synth.CONFIGS[3], name="qkv-forms", n_layers=1, hidden=H, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=d, ffn=512,
                         vocab=2048, ad_heads=n_q if H % n_q == 0 else 4, seed=23)
    dev_w = clover.upload_weights(synth.WeightStore(shape))
    rng = np.random.default_rng(M)
    parent = np.array([-1] + sorted(int(rng.integers(max(0, u // 3 - 2), u)) for u in range(1, nodes)), np.int32)
    rank = np.zeros(nodes, np.int32)
    for u in range(1, nodes):
        rank[u] = sum(parent[v] == parent[u] for v in range(1, u))
    lens = [int(v) for v in rng.integers(0, 70, batch)]
    max_seq = (max(lens) + 2 * R + 63) // 32 * 32
    pages = rng.permutation(batch * max_seq // 32).astype(np.int32)
    tok = torch.randint(0, shape.vocab, (batch, R), generator=torch.Generator().manual_seed(1)).int()
    return shape, dev_w, parent, rank, lens, max_seq, pages, tok


def _compare(H, n_q, n_kv, d, batch, nodes, R):
    """One layer by the MFMA path and by the fp32-ALU kernels.  Returns whether the former's attention is the MFMA one too, and the launches
    of its QKV projection and of the rotation behind it."""
    shape, dev_w, parent, rank, lens, max_seq, pages, tok = _model(H, n_q, n_kv, d, batch, nodes, R)
    import torch
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, parent, rank, batch, max_seq, R, flags=flags | (clover.FLAG_INTERVAL_MASK if R > 128 else 0))
        if flags == 0:
            path = g.path_info()
            assert path & 1
            g.set_page_table(pages)
        g.set_seq_len(lens, [max(v - 1, 0) for v in lens])
        for b in range(batch):                                 # (the cached rows: zeros)
            if lens[b]:
                g.write_kv(0, 0, b, 0, np.zeros((lens[b], n_kv, d), np.float32), np.zeros((lens[b], n_kv, d), np.float32))
        g.tree_tokens.copy_(tok)
        g.profile_enable(flags == 0)
        g.verify_tree(batch)
        torch.cuda.synchronize()
        if flags == 0:
            ran = g.profile_collect()
        assert list(g.seq_len()) == lens                       # (no guard fired)
        # every slot: those behind the nodes stay as they were, zeros on the MFMA path
        kv = [g.read_kv(0, 0, b, 0, max_seq if flags == 0 else lens[b] + nodes) for b in range(batch)]
        out.append((kv, g.hidden[:, :nodes].double().cpu()))
        g.close()
    tol = _tolerance(H)
    for b in range(batch):
        for got, want in zip(out[0][0][b], out[1][0][b]):
            new = slice(lens[b], lens[b] + nodes)
            assert np.abs(got[new] - want[new]).max() <= tol, (b, np.abs(got[new] - want[new]).max(), tol)
            assert not got[:lens[b]].any() and not got[lens[b] + nodes:].any()
    # the rows' results through attention and FFN (the bound of the attention's tests; keys and values of another scale with H)
    assert (out[0][1] - out[1][1]).abs().max().item() <= 2e-3 * max(1.0, H / 1024)
    return bool(path & 2), ran["gemm_qkv"][1], ran["rope_kv_write"][1]


def _tolerance(H):
    """of keys and values: products of normalised rows and N(0, 0.02) weights, 16 mantissa bits on one side (the bound of the GEMM's own
    tests), turned by an angle, and once more 2^-17 of a value of up to 5 sigma"""
    return 4e-5 * np.sqrt(H) * 0.02 * 4 * 1.5 + 2.0 ** -17 * 5 * 0.02 * np.sqrt(H)


@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_kv,d,batch,nodes,R,ranges,launches", CASES)
def test_keys_and_values(H, n_q, n_kv, d, batch, nodes, R, ranges, launches):
    import torch   # (in front of the library, which then finds torch's HIP runtime)
    assert torch.cuda.is_available()
    assert _ranges((batch - 1) * R + nodes, (n_q + 2 * n_kv) * d, H) == ranges
    assert _compare(H, n_q, n_kv, d, batch, nodes, R) == (True, 1, launches - 1)


# Heads of 64, and groups of seven, three and five heads, which the MFMA attention does not take: two launches up to 32 rows, one above, over
# one to eight ranges of K on one XCD and on several, by tiles of 64 to 256 rows, the last of them not whole, whose results are finished
# two blocks, a row of blocks or a part of a row of blocks at a time.
WITHOUT_MFMA_ATTENTION = [(1024, 6, 3, 64, 1, 1, 1), (896, 7, 1, 128, 1, 17, 17), (2560, 20, 4, 128, 1, 24, 24), (256, 4, 1, 64, 2, 16, 16),
                          (1024, 6, 3, 64, 1, 33, 33), (256, 4, 4, 64, 2, 40, 41), (2048, 32, 8, 64, 2, 47, 50), (1024, 16, 2, 64, 7, 19, 23),
                          (2048, 32, 8, 64, 4, 90, 100), (3584, 28, 4, 128, 1, 64, 64), (2304, 36, 9, 64, 1, 97, 97), (3584, 28, 4, 128, 3, 99, 101),
                          (1152, 9, 3, 128, 1, 130, 133), (2432, 38, 38, 64, 1, 130, 133), (3840, 32, 8, 64, 3, 99, 100),
                          (5120, 28, 4, 128, 2, 250, 256), (1024, 28, 4, 128, 8, 250, 256), (2432, 38, 38, 64, 8, 250, 256),
                          (1024, 6, 3, 64, 7, 19, 23), (256, 4, 1, 64, 1, 12, 12)]


@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_kv,d,batch,nodes,R", WITHOUT_MFMA_ATTENTION)
def test_keys_and_values_without_mfma_attention(H, n_q, n_kv, d, batch, nodes, R):
    rows = (batch - 1) * R + nodes
    assert _compare(H, n_q, n_kv, d, batch, nodes, R) == (False, 1, 1 if rows <= 32 else 0)


# Tiles of 32, 64, 128, 160 and 256 rows (those of 160 and more request what they need only behind the meeting); ranges on one XCD, and
# six of them on several; heads with and without MFMA attention.
LEAVING = [(1024, 8, 2, 128, 1, 5, 5), (4096, 32, 8, 128, 2, 30, 33), (3072, 24, 24, 128, 4, 27, 28), (2304, 36, 9, 64, 1, 97, 97),
           (2432, 38, 38, 64, 1, 130, 133), (5120, 28, 4, 128, 2, 250, 256)]


@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_kv,d,batch,nodes,R", LEAVING)
def test_members_that_leave(H, n_q, n_kv, d, batch, nodes, R):
    """Workgroups that look at the meeting's word once or not at all leave their share to the last one.  A share is summed in the order
    of the ranges whoever does it, so that no bit of the results changes, pass after pass in the same words."""
    shape, dev_w, parent, rank, lens, max_seq, pages, tok = _model(H, n_q, n_kv, d, batch, nodes, R)
    import torch
    set_polls = clover.load_library()._ZN3clv14set_meet_pollsEP10clover_ctxi
    set_polls.restype, set_polls.argtypes = None, [C.c_void_p, C.c_int]
    out = []
    for polls in (None, 0, 1):
        g = clover.Clover(shape, dev_w, parent, rank, batch, max_seq, R, flags=clover.FLAG_INTERVAL_MASK if R > 128 else 0)
        g.set_page_table(pages)
        if polls is not None:
            set_polls(g.ctx, polls)
        g.set_seq_len(lens, [max(v - 1, 0) for v in lens])
        for b in range(batch):
            if lens[b]:
                g.write_kv(0, 0, b, 0, np.zeros((lens[b], n_kv, d), np.float32), np.zeros((lens[b], n_kv, d), np.float32))
        got = []
        for i in range(3):                                     # (other tokens: nothing that is left of the pass before is right)
            g.tree_tokens.copy_((tok + i) % shape.vocab)
            g.profile_enable(True)
            g.verify_tree(batch)
            torch.cuda.synchronize()
            ran = g.profile_collect()
            assert (ran["gemm_qkv"][1], ran["rope_kv_write"][1]) == (1, 0)
            got.append(g.hidden[:, :nodes].cpu().numpy())
            got += [v for b in range(batch) for v in g.read_kv(0, 0, b, 0, max_seq)]
        assert list(g.seq_len()) == lens
        out.append(got)
        g.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_kv,d", [(1024, 6, 3, 64), (896, 7, 1, 128)])
def test_prompts_without_mfma_attention(H, n_q, n_kv, d):
    """one range of K, in tiles of many rows, the last of them with a part of its rows; the last row's result rests on its q as well"""
    import torch
    assert torch.cuda.is_available()
    n = 553
    shape = synth.scaled(synth.CONFIGS[3], name="qkv-prompt", n_layers=1, hidden=H, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=d, ffn=512, vocab=2048,
                         ad_heads=4, seed=29)
    dev_w = clover.upload_weights(synth.WeightStore(shape))
    parent, rank = np.array([-1, 0, 0], np.int32), np.array([0, 0, 1], np.int32)
    tok = torch.randint(0, shape.vocab, (n,), generator=torch.Generator().manual_seed(3)).int().cuda()
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, parent, rank, 1, 640, 64, flags=flags, prefill_rows=256)
        g.prefill_prompt(0, tok)
        torch.cuda.synchronize()
        if flags == 0:
            assert g.path_info() == 1
        out.append((*g.read_kv(0, 0, 0, 0, n), g.hid_acc[0, 0].double().cpu().numpy()))
        g.close()
    for got, want, tol in zip(*out, (_tolerance(H), _tolerance(H), 2e-3 * max(1.0, H / 1024))):
        assert np.abs(got - want).max() <= tol, (np.abs(got - want).max(), tol)


def test_what_one_launch_takes():
    """The rule over widths, heads and row counts: workgroups that exchange partial tiles in front of the MFMA attention share an XCD and one row
    tile, and no launch has more tiles than there are meetings."""
    import torch   # noqa: F401 (in front of the library)
    taken = 0
    for H in range(256, 8193, 256):
        for n_q, n_kv, d in {(H // 128, H // 128, 128), (H // 128, max(1, H // 512), 128), (H // 64, max(1, H // 256), 64), (28, 4, 128), (40, 8, 128), (7, 1, 128)}:
            if n_q % n_kv:
                continue
            N, mfma = (n_q + 2 * n_kv) * d, d == 128 and n_q // n_kv in (1, 2, 4, 8)
            for M in (1, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 160, 256, 512, 1000, 2048):
                ranges = _ranges(M, N, H)
                one, (rb, wb, row_tiles, kp, stages) = _joins(M, N, H, ranges, mfma)
                if not one:
                    continue
                taken += 1
                assert kp == ranges
                tiles = -(-N // 16 // wb)
                assert kp == 1 or tiles * row_tiles <= 256
                if mfma:
                    assert 2 <= kp <= 4 and row_tiles == 1 and rb <= 4 and -(-tiles // 8) * kp <= 32, (H, n_q, n_kv, M, rb, wb, row_tiles, kp)
                    assert M <= 32 or kp >= 3
                    assert M <= 64 or (M <= 128 and stages >= 16)
                else:
                    assert M > 32
    assert taken > 500, taken
