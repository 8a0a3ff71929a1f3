"""The robustness adjoint's sums over output tiles, at the ends of their range:
alignment tiles cut by the frame's edge, blocks narrower than eight cells, an
alignment tile with more than 64 output tiles, and one with several blocks."""
import numpy as np
import pytest
import torch

import oracle.adjoint as oa
from test_gpu_backward import check, gpu_backward, grad_case

pytestmark = pytest.mark.gpu

# the same per-entry bound as the adjoint's other tests (`check`)
CASES = [dict(scale=3.0, seed=21, n=2, h=64, w=66, tile=64),     # 24 x 3 output tiles in the first one
         dict(scale=3.0, seed=22, n=2, h=66, w=72, tile=64, ref=1),
         dict(scale=1.0, seed=23, n=3, h=36, w=50, tile=32),     # blocks of 2 rows and 1 column
         dict(scale=1.25, seed=24, n=2, h=44, w=52, tile=8),
         dict(scale=2.5, seed=25, n=2, h=34, w=40, tile=8),
         dict(scale=1.0, seed=26, n=2, h=34, w=34, tile=64)]     # one alignment tile, cut


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_tile_sums_match_oracle_adjoint(case):
    print("[case]", case, flush=True)
    f, m, d, t, g_out = grad_case(**case)
    want_t, want_m = oa.merge_backward(f, m, d, t, g_out)
    first = None
    for _ in range(3):   # the tuning sums' finishing workgroup differs from run to run
        got_t, got_m = gpu_backward(f, m, d, t, g_out)
        first = first or (got_t, got_m)
        assert np.array_equal(got_t, first[0]) and np.array_equal(got_m, first[1])
    check(got_t, want_t, "tuning gradient")
    check(got_m, want_m, "motion gradient")
    assert np.all(got_m[d.ref_frame] == 0.0)
    torch.cuda.synchronize()


# A cell of R_hat is read by 4 * scale output rows, which lie in up to three of
# the adjoint's tiles of eight rows at scale 4 and up to five at scale 8.
HIGH_SCALES = [dict(scale=4.0, seed=31, n=2, h=34, w=40, tile=8),
               dict(scale=4.5, seed=32, n=3, h=34, w=40, tile=16, ref=1),
               dict(scale=5.0, seed=33, n=2, h=40, w=34, tile=8, cfa=1),
               dict(scale=6.7, seed=34, n=2, h=34, w=40, tile=16),
               dict(scale=7.3, seed=35, n=3, h=36, w=34, tile=8, cfa=2),
               dict(scale=8.0, seed=36, n=2, h=34, w=36, tile=32, ref=1)]


@pytest.mark.parametrize("case", HIGH_SCALES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_cells_of_many_output_tiles(case):
    print("[case] high scale", case, flush=True)
    f, m, d, t, g_out = grad_case(**case)
    want_t, want_m = oa.merge_backward(f, m, d, t, g_out)
    got_t, got_m = gpu_backward(f, m, d, t, g_out)
    check(got_t, want_t, "tuning gradient")
    check(got_m, want_m, "motion gradient")
