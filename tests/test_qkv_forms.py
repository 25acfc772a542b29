"""The QKV projection's launch, which also rotates, writes q and fills the caches: its tiles over one and several ranges of K, whole and
partial row blocks and last tiles, sequences with unused rows between them, both head sizes, shuffled pages.  Reference: the
fp32-ALU kernels of the same model."""
import ctypes as C

import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu
# (hidden, query heads, KV heads, head size, sequences, nodes, rows of a sequence, K ranges that the rule takes)
CASES = [(4096, 32, 8, 128, 1, 1, 1, 8), (4096, 32, 8, 128, 1, 16, 24, 8), (4096, 32, 8, 128, 1, 17, 17, 8), (4096, 32, 8, 128, 2, 30, 33, 4),
         (4096, 32, 8, 128, 3, 32, 32, 4), (4096, 32, 8, 128, 1, 120, 128, 4), (4096, 32, 8, 128, 8, 32, 32, 4),
         (1024, 8, 2, 128, 1, 5, 5, 4), (1024, 8, 2, 128, 3, 50, 60, 4), (1024, 6, 3, 64, 1, 33, 33, 4), (1024, 6, 3, 64, 7, 19, 23, 4),
         (640, 5, 5, 128, 2, 9, 40, 2), (256, 4, 1, 64, 1, 12, 12, 1), (512, 32, 32, 128, 12, 50, 51, 1), (2048, 16, 16, 128, 9, 60, 60, 1)]


@pytest.mark.parametrize("H,n_q,n_kv,d,batch,nodes,R,ranges", CASES)
def test_keys_and_values(H, n_q, n_kv, d, batch, nodes, R, ranges):
    import torch
    lib = clover.load_library()
    M, N, form = (batch - 1) * R + nodes, (n_q + 2 * n_kv) * d, (C.c_int32 * 5)()
    assert lib.clover_op_gemm_form(0, M, N, H, ranges, form) == 0
    print(f"qkv M={M} N={N} K={H} form={list(form)}", flush=True)
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
    out = []
    for flags in (0, clover.FLAG_GENERIC):
        g = clover.Clover(shape, dev_w, parent, rank, batch, max_seq, R, flags=flags)
        if flags == 0:
            assert g.path_info() & 1
            g.set_page_table(pages)
        g.set_seq_len(lens, [max(v - 1, 0) for v in lens])
        for b in range(batch):                                 # (the cached rows: zeros)
            if lens[b]:
                g.write_kv(0, 0, b, 0, np.zeros((lens[b], n_kv, d), np.float32), np.zeros((lens[b], n_kv, d), np.float32))
        g.tree_tokens.copy_(tok)
        g.verify_tree(batch)
        torch.cuda.synchronize()
        assert list(g.seq_len()) == lens                       # (no guard fired)
        # every slot: those behind the nodes stay as they were, zeros on the MFMA path
        kv = [g.read_kv(0, 0, b, 0, max_seq if flags == 0 else lens[b] + nodes) for b in range(batch)]
        out.append((kv, g.hidden[:, :nodes].double().cpu()))
        g.close()
    # products of normalised rows and N(0, 0.02) weights, 16 mantissa bits on one side (the bound of the GEMM's own tests), turned
    # by an angle, and once more 2^-17 of a value of up to 5 sigma
    tol = 4e-5 * np.sqrt(H) * 0.02 * 4 * 1.5 + 2.0 ** -17 * 5 * 0.02 * np.sqrt(H)
    for b in range(batch):
        for got, want in zip(out[0][0][b], out[1][0][b]):
            new = slice(lens[b], lens[b] + nodes)
            assert np.abs(got[new] - want[new]).max() <= tol, (b, np.abs(got[new] - want[new]).max(), tol)
            assert not got[:lens[b]].any() and not got[lens[b] + nodes:].any()
    # the rows' results through attention and FFN (the bound of the attention's tests; keys and values of another scale with H)
    assert (out[0][1] - out[1][1]).abs().max().item() <= 2e-3 * max(1.0, H / 1024)
