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

import oracle.align as oa

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


def coherent_frames(h, w, seed):
    """A base frame of 0 to 3 and a frame of 65535 less 0 to 3 (periodic over
    eight) per 16 x 16 raw pixels, a level-3 pixel: every candidate of a level-3
    block costs about 2^54, and the candidates differ by the correlation of the
    small terms, a few units."""
    rng = np.random.default_rng(seed)
    ph, pw = -(-h // 16), -(-w // 16)
    r = np.tile(rng.integers(0, 4, (8, 8)), (ph // 8 + 1, pw // 8 + 1))[:ph, :pw]
    f = np.zeros((2, ph * 16, pw * 16), np.uint16)
    f[0, ::16, ::16] = rng.integers(0, 4, (ph, pw))
    f[1] = 65535
    f[1, ::16, ::16] = 65532 + r
    return np.ascontiguousarray(f[:, :h, :w])


@pytest.mark.parametrize("levels,radius", [(4, 4), (5, 2)])   # level 3 the coarsest, and below another
def test_costs_beyond_float64(levels, radius):
    """Level-3 costs above 2^53 that float64 cannot tell apart: the sums over
    the pieces have to be 64-bit integers."""
    h, w, seed = 520, 536, 1
    f = coherent_frames(h, w, seed)
    d = synth.Desc(2, h, w, tile_size=16, black_level=0.0, white_level=65535.0, noise_a=1e-4, noise_b=1e-6)
    params = {"levels": levels, "gate": 0.0, "lk_iterations": 0}
    base, img = (oa.pyramid(oa.quad_sums(x), levels, 8) for x in f)
    guess = np.zeros(oa.block_grid(base[3].shape, 8) + (2,), dtype=np.int64)
    if levels == 5:
        coarse = np.zeros(oa.block_grid(base[4].shape, 8) + (2,), dtype=np.int64)
        guess = oa.upsample_guess(oa.match_level(base[4], img[4], 8, coarse, 4), 8, base[3].shape, 8)
    vec = oa.match_level(base[3], img[3], 8, guess, radius)
    largest, other = 0, 0
    for by, bx in np.ndindex(vec.shape[:2]):
        ys, xs = np.arange(8 * by, min(8 * by + 8, base[3].shape[0])), np.arange(8 * bx, min(8 * bx + 8, base[3].shape[1]))
        keys = []
        for dy in range(-radius, radius + 1):
            for dx in range(-radius, radius + 1):
                u = guess[by, bx] + (dx, dy)
                e = img[3][np.ix_(np.clip(ys + u[1], 0, img[3].shape[0] - 1), np.clip(xs + u[0], 0, img[3].shape[1] - 1))]
                e = e - base[3][np.ix_(ys, xs)]
                largest = max(largest, int((e * e).sum()))
                keys.append((sum(float((q * q).sum()) for q in e), dx * dx + dy * dy, len(keys), *u))   # float64 over the rows
        other += tuple(vec[by, bx]) != min(keys)[3:]
    assert largest > 2 ** 53 and other > 0   # float64 would decide some block otherwise
    check_full(f, d, params, what=f"coherent {levels} levels")
