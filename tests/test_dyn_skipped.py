"""A sequence that the first draft call skips (m = 0) in a workspace whose memory held anything: its dynamic tables are read
along with the others', so they must name candidates that exist, and the other sequence's tree must not depend on them."""
import numpy as np
import pytest

from paper_2408_00264_amd import clover, synth
from tests.test_gpu_parity import MINI, TINY

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", ["fp32", "bf16", "bf16_generic"])
@pytest.mark.parametrize("skipped", [0, 1])
def test_skipped_sequence(case, skipped, monkeypatch):
    import torch
    shape = MINI if "bf16" in case else TINY
    w = clover.upload_weights(synth.WeightStore(shape))
    new, out = torch.empty, []
    for byte in (0, 0x7f):
        with monkeypatch.context() as mp:
            mp.setattr(torch, "empty", lambda *a, **k: new(*a, **k).fill_(byte) if k.get("dtype") == torch.uint8 else new(*a, **k))
            g = clover.Clover(shape, w, np.array([-1], np.int32), np.array([0], np.int32), 2, 128, 24,
                              flags=clover.FLAG_GENERIC if "generic" in case else 0)
        g.set_dynamic_tree(16, 4, 3)
        b = 1 - skipped
        g.prefill_prompt(b, torch.arange(5, 25, dtype=torch.int32, device="cuda"))
        g.m.fill_(1)
        g.m[skipped] = 0
        for _ in range(2):
            g.draft_tree(2)
            tree = g.read_dynamic_tree(b)
            out.append([g.tree_tokens[b, :16].cpu().numpy(), tree["parent"], tree["keep"], g.m.cpu().numpy()])
            g.verify_tree(2)
            g.accept_and_compact(2)
            g.m[skipped] = 0
        torch.cuda.synchronize()
    half = len(out) // 2
    for a, c in zip(out[:half], out[half:]):
        for x, y in zip(a, c):
            assert np.array_equal(x, y), (x, y)
