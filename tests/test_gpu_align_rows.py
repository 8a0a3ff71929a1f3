"""Block matching by rows and Lucas-Kanade by columns at the sizes where they
can go wrong: blocks of 8, 16 and 32 with remainders in both directions, block
counts that do not fill a wave, radius 2 and 4 on every level that takes them
(levels 0-2 in float64, level 3 in 64-bit integers, level 4 and other radii by
the general kernel), windows of 16, 32 and 64 columns clipped on every side,
and values that alternate between 0 and 65535, whose costs are the largest a
16-bit burst can have. Block-matching vectors are integers and must be equal;
refined vectors are compared as in test_gpu_align (float32 rounding of the
result, float64 sums)."""
import numpy as np
import pytest

from paper_1905_03277_amd import synth
from test_gpu_align import check_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,tile,ref,params", [
    (3, 130, 158, 16, 0, {"levels": 1, "radius_coarse": 2}),   # 9 x 10 blocks of 8 on one level, the last ones ragged
    (3, 130, 158, 16, 1, {"levels": 1, "radius_coarse": 4}),
    (3, 132, 146, 16, 2, {"levels": 3}),                       # radius 4 in float64 on level 2
    (2, 264, 280, 16, 0, {"levels": 4}),                       # radius 4 in integers on level 3
    (2, 520, 536, 16, 1, {"levels": 5}),                       # level 4 general, radius 2 in integers on level 3
    (3, 130, 158, 32, 0, {"radius_fine": 2}),
    (2, 194, 206, 64, 1, {"radius_fine": 2}),
    (2, 130, 158, 32, 0, {"radius_fine": 3, "radius_coarse": 5}),   # radii that take the general kernel
])
@pytest.mark.parametrize("extreme", [False, True])
def test_rows_and_columns(n, h, w, tile, ref, params, extreme):
    if extreme:
        rng = np.random.default_rng(8100 + h + tile)
        cells = rng.integers(0, 2, size=(n, h // 2, w // 2)).astype(np.uint16) * np.uint16(65535)
        f = np.ascontiguousarray(cells.repeat(2, axis=1).repeat(2, axis=2))   # whole quads at 0 or 65535
        d = synth.Desc(n, h, w, tile_size=tile, black_level=0.0, white_level=65535.0, noise_a=1e-4, noise_b=1e-6)
        params = dict(params, lk_iterations=1)   # noise against noise: one step keeps the vectors in range
    else:
        b = synth.make_burst(n, h, w, seed=8000 + h + tile, tile_size=tile, scene="texture", sigma_t=3.0)
        f, _ = b.numpy()
        d = b.desc
    check_full(f, d.replace(ref_frame=ref), params, what=f"{n}x{h}x{w} t{tile} extreme={extreme}")
