"""The token a verification emits, for crafted rows of logits: the argmax of a row and the draw at a temperature > 0.
The rows go through the public calls on a model whose weights play no part (single-node trees, one row per sequence)."""
import numpy as np
import pytest

from oracle import clover2_oracle as O
from paper_2408_00264_amd import clover, synth

pytestmark = pytest.mark.gpu


def _context(vocab, batch, parent=(-1,), rank=(0,)):
    import torch
    shape = synth.scaled(synth.CONFIGS[1], vocab=vocab, hidden=64, n_q_heads=1, n_kv_heads=1, ffn=64)
    weights = {n: torch.zeros(s, dtype=torch.float32, device="cuda") for n, s in synth.weight_shapes(shape).items()}
    return torch, clover.Clover(shape, weights, np.asarray(parent, np.int32), np.asarray(rank, np.int32), batch, 32, len(parent))


def argmax_rows(V):
    """rows whose largest value lies at the edges of pieces, lanes and 2048-wide chunks; equals; values that order oddly"""
    rng = np.random.default_rng(V)
    rows = [rng.standard_normal(V) for _ in range(3)]
    for at in {0, V - 1, min(2047, V - 1), min(2048, V - 1), V // 2}:
        rows.append(rng.standard_normal(V))
        rows[-1][at] = 9.0
    rows.append(np.full(V, 1.5))                                 # all equal: the lowest id
    for a, b in ((5, 9), (1, V - 1), (V // 2, V - 2), (min(2046, V - 2), V - 1)):   # two equal maxima, ids a < b
        rows.append(rng.standard_normal(V))
        rows[-1][[a, b]] = 9.0
    rows.append(np.where(np.arange(V) == 7, -0.0, np.where(np.arange(V) == 11, 0.0, -1.0)))   # -0 and +0 are equals
    rows.append(np.full(V, -np.finfo(np.float32).max))           # a mask's lowest value everywhere
    rows.append(np.full(V, -np.inf))
    rows.append(np.where(np.arange(V) == V - 3, -3e38, -np.inf))
    rows.append(np.where(np.arange(V) == 6, np.inf, 0.0))
    rows = np.asarray(rows, np.float32)
    bits = np.full((2, V), 0xFFFFFFFF, np.uint32)                # the NaN of all ones: alone, and below one number
    bits[1, V - 2] = np.float32(-1e30).view(np.uint32)
    return np.concatenate([rows, bits.view(np.float32)])


@pytest.mark.parametrize("V", [16, 1024, 2048, 2052, 5004, 5003, 128256])   # (5003: not a multiple of the 16-byte piece)
def test_argmax_of_crafted_rows(V):
    rows = argmax_rows(V)
    torch, g = _context(V, len(rows))
    print(f"argmax of {len(rows)} rows, vocabulary {V}", flush=True)
    g.logits[:, 0].copy_(torch.from_numpy(rows.view(np.int32)).cuda().view(torch.float32))   # (as bits: NaNs stay what they are)
    g.accept_and_compact(len(rows))
    got = g.new_tokens[:, 0].cpu().numpy()
    # the order of the library: by value, -0 = +0, a NaN of negative sign below everything; the lowest id among equals
    with np.errstate(invalid="ignore"):
        u = (rows + np.float32(0)).view(np.uint32)
    u = np.where(np.isnan(rows), rows.view(np.uint32), u)
    key = np.where(u >> 31, ~u, u | np.uint32(1 << 31))
    np.testing.assert_array_equal(got, key.argmax(1))
    assert g.m.cpu().tolist() == [1] * len(rows)


def draw_rows(V):
    """(tokens and their log-masses, uniform): the draw must land in the middle of a step of the cumulative sum, or, with
    the uniform 0, on the first token that has any mass, however small beside the rest"""
    at = lambda t: min(t, V - 1)
    quarters = [3, at(63 * 2048 + 5), at(64 * 2048 + 7), V - 1]          # chunks 0, 63, 64 and the last one
    cases = [({t: np.log(0.25) for t in quarters}, u) for u in (0.1, 0.4, 0.6, 0.9, 0.0, 1.0 - 2.0 ** -24)]
    t = at(2048) if V > 4096 else 0                                      # one chunk: neighbours, another thread, wavefront
    fifths = [t + d for d in (0, 1, 9, 600, 1023) if t + d < V]
    cases += [({f: np.log(0.2) for f in fifths}, u) for u in (0.1, 0.3, 0.5, 0.7, 0.9, 0.0, 1.0 - 2.0 ** -24)]
    for tiny, big in ((0, V - 1), (5, V // 2), (t + 3, t + 700), (t, t + 1), (t + 2, at(t + 130 * 2048))):
        if tiny < big < V:
            cases.append(({tiny: -50.0, big: 0.0}, 0.0))                 # the step at the small token holds the target
            cases.append(({tiny: -50.0, big: 0.0}, 0.5))
    return cases


@pytest.mark.parametrize("V", [1024, 5004, 5003, 128256, 200002, 262144])
@pytest.mark.parametrize("floor", [-1e4, -np.inf], ids=["finite", "masked"])
def test_draw_from_crafted_rows(V, floor):
    cases = draw_rows(V)
    torch, g = _context(V, len(cases))
    print(f"draw from {len(cases)} rows, vocabulary {V}", flush=True)
    rows = np.full((len(cases), V), floor, np.float32)
    uni = np.zeros((len(cases), 1, 17), np.float32)
    for i, (mass, u) in enumerate(cases):
        for t, z in mass.items():
            rows[i, t] = z
        uni[i, 0, 16] = u
    g.logits[:, 0].copy_(torch.from_numpy(rows).cuda())
    g.accept_and_compact_sampled(len(cases), 1.0, torch.from_numpy(uni).cuda())
    got = g.new_tokens[:, 0].cpu().numpy().tolist()
    want = [O.accept_sampled([0], rows[i:i + 1].astype(np.float64), [-1], 1.0, uni[i].astype(np.float64))[1] for i in range(len(cases))]
    assert got == want, [(c, a, b) for c, a, b in zip(cases, got, want) if a != b]
