"""The base frame's sum behind the SNR: one partial sum per workgroup in host
memory. Sizes at one workgroup, its edge, and past the most there are, in turn
on one library state, so that a partial sum left by a larger frame would show."""
import numpy as np
import pytest
import torch

import oracle.noise as on
from paper_1905_03277_amd import synth, torch_ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(4, 4), (64, 64), (64, 66), (2048, 2050), (4, 4), (4, 2050)]])
def test_snr_is_that_of_the_exact_sum(shapes):
    rng = np.random.default_rng(3)
    base = synth.make_burst(2, 4, 4, seed=3).desc
    for h, w in shapes:
        f = rng.integers(0, 65536, size=(2, h, w), dtype=np.uint16)
        d = base.replace(height=h, width=w, ref_frame=1, white_level=65535.0)
        print("[case] frame sum", h, w, flush=True)
        _, _, snr = torch_ops.auto_tuning(torch.from_numpy(f.view(np.int16)).to("cuda:0"), d)
        assert snr == on.frame_snr(f[1], d.noise_a, d.noise_b, d.black_level, d.white_level)
