"""The batch's fused statistics launch: a graph captured without the LDS of the
detail term S.3 is not replayed with it."""
import pytest
import torch

from paper_1905_03277_amd import synth, torch_ops

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_detail_term_switched_on_between_replays():
    """hf_ratio 0 -> positive -> 0 with unchanged shapes: the statistics of S.3 need LDS the first graph's
    launch does not have."""
    b = synth.make_burst(3, 64, 96, seed=9300)
    f, m = b.frames.to(DEV), b.motion.to(DEV)
    for hf in (0.0, 0.5, 0.0, 0.5):
        t = b.tuning.replace(hf_ratio=hf)
        want = torch_ops.merge(f, m, b.desc, t)
        got = torch_ops.merge_batch([(f, m, b.desc, t)])[0]
        torch.cuda.synchronize()
        print("[case] hf_ratio", hf, flush=True)
        assert torch.equal(got, want)
