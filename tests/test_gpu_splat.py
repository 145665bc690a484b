"""The renderer's staging and splat at the sizes where they change form, against
the binary32 mirror bit for bit (pixel sums are exact integers)."""

import numpy as np
import pytest

pytest.importorskip("torch")
import torch  # noqa: E402

import gpu_util as gu  # noqa: E402
import paper_2512_09664_amd as sp  # noqa: E402
from oracle import ra32 as ra  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(H, W, n, d_range, tile, seed, box=None):
    rng = np.random.default_rng([seed, n, H, W])
    x0, x1, y0, y1 = box or (-3.0, W + 3.0, -3.0, H + 3.0)
    q = {"x": rng.uniform(x0, x1, n), "y": rng.uniform(y0, y1, n), "z": rng.uniform(-1, 1, n),
         "d": rng.uniform(*d_range, n), "I0": rng.uniform(0.05, 0.2, n)}
    q = {k: v.astype(np.float32) for k, v in q.items()}
    x2, y2 = (q[k] + rng.uniform(-2, 2, n).astype(np.float32) for k in ("x", "y"))
    b = gu.batch_for([(H, W)], [(4, 4)], [n])
    t = {k: gu.to_dev(v) for k, v in q.items()}
    rp = sp.render_params(0.5, 16.0 if d_range[1] > 8 else 8.0, 0, 0.7, 0.0, 0)
    img = sp.render_pair(b, t["x"], t["y"], gu.to_dev(x2), gu.to_dev(y2), t["z"], t["d"], t["I0"], rp,
                         sp.tiling(*tile))
    torch.cuda.synchronize()
    got = gu.to_np(img).reshape(2, H, W)
    for f, (xx, yy) in enumerate(((q["x"], q["y"]), (x2, y2))):
        assert np.array_equal(got[f], ra.render(xx, yy, q["z"], q["d"], q["I0"], H, W, 0.5)), f


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 600])
@pytest.mark.parametrize("tile", [(64, 32, 2048, 64), (64, 32, 2048, 64, 1)])
def test_list_lengths(n, tile):
    """One tile's list: 1, 2 and 4 lanes per particle, one pass and several."""
    _check(32, 64, n, (1.0, 5.0), tile, 1, box=(8.0, 56.0, 8.0, 24.0))


@pytest.mark.parametrize("d", [(0.2, 1.2), (1.0, 2.0), (1.8, 2.7), (2.5, 3.4), (3.2, 4.0), (3.9, 5.4), (5.2, 6.7),
                               (6.5, 16.0)])
@pytest.mark.parametrize("tile", [(8, 8, 256, 32), (64, 64, 2048, 128)])
def test_patch_widths(d, tile):
    """Every width class of the column factors, whole patches and patches cut by
    tiles far smaller than them; 8 x 8 tiles make a grid that fills the chip
    (fewest lanes per particle), 64 x 64 tiles one that does not."""
    _check(190, 186, 700, d, tile, 2)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 129, 513, 600])
@pytest.mark.parametrize("d", [(3.9, 4.4), (4.2, 5.4), (5.2, 7.0)])
def test_wide_lists(n, d):
    """Wide patches in one tile's list: up to two lanes' worth, one wave's worth and
    more particles, with particles left over at every step of it."""
    _check(64, 64, n, d, (64, 64, 2048, 128), 3, box=(8.0, 56.0, 8.0, 56.0))


@pytest.mark.parametrize("d,d_max", [((0.8, 1.2), 1.5), ((1.0, 3.0), 3.0), ((2.0, 5.0), 5.0), ((3.0, 7.0), 7.0),
                                     ((6.0, 16.0), 16.0), ((1.0, 4.0), 16.0)])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16), (32, 32), (64, 16), (64, 32), (128, 32), (64, 64)])
@pytest.mark.parametrize("persistent", [0, 1])
def test_tiles_and_diameter_bounds(tile, d, d_max, persistent):
    """Every tile shape with diameter bounds on both sides of the row walk's change of
    form, lists of one and of several passes, patches cut by tile and image edges."""
    H, W, n = 150, 186, 420
    rng = np.random.default_rng([int(10 * d_max), tile[0], tile[1]])
    q = {"x": rng.uniform(-3, W + 3, n), "y": rng.uniform(-3, H + 3, n), "z": rng.uniform(-1, 1, n),
         "d": rng.uniform(*d, n), "I0": rng.uniform(0.01, 0.05, n)}
    q["x"][:200], q["y"][:200] = rng.uniform(60, 72, 200), rng.uniform(60, 72, 200)
    q = {k: v.astype(np.float32) for k, v in q.items()}
    b = gu.batch_for([(H, W)], [(4, 4)], [n])
    t = {k: gu.to_dev(v) for k, v in q.items()}
    rp = sp.render_params(0.5, d_max, 0, 0.7, 0.0, 0)
    img = sp.render_pair(b, t["x"], t["y"], t["x"], t["y"], t["z"], t["d"], t["I0"], rp,
                         sp.tiling(*tile, 256, 64, persistent))
    got = gu.to_np(img).reshape(2, H, W)
    want = ra.render(q["x"], q["y"], q["z"], q["d"], q["I0"], H, W, 0.5)
    assert np.array_equal(got[0], want) and np.array_equal(got[1], want)


def test_wide_patches_on_small_tiles_cost():
    """Patches that fill a tile's rows do not add to the same words in step: with d to 16,
    32 x 32 tiles take at most half as long again as 64 x 64 ones."""
    n, side = 16, 512
    b = gu.batch_for([(side, side)] * n, [(4, 4)] * n, [13107] * n)
    gen = torch.Generator(device=gu.DEV).manual_seed(1)
    u = lambda lo, hi: lo + (hi - lo) * torch.rand(b.n_particles, generator=gen, device=gu.DEV)  # noqa: E731
    x, y, z, d, I0 = u(0, side), u(0, side), u(-1, 1), u(4.0, 16.0), u(0.001, 0.002)
    rp = sp.render_params(0.5, 16.0, 1, 0.7, 0.0, 12)
    best = {}
    for tile in ((64, 64), (32, 32)):
        tl = sp.tiling(*tile, 2048, 64)
        ws = sp.alloc_workspace(b, rp, tl)
        for _ in range(6):
            sp.timing_read(None)
            sp.timing_enable(True)
            sp.render_pair(b, x, y, y, x, z, d, I0, rp, tl, workspace=ws)
            torch.cuda.synchronize()
            sp.timing_enable(False)
            best[tile] = min(best.get(tile, 1e9), sp.timing_read("render_tile")[0])
    sp.timing_read(None)
    assert best[(32, 32)] <= 1.5 * best[(64, 64)], best


@pytest.mark.parametrize("blur", [0, 1, 2, 3])
def test_wide_patches_on_default_tiles(blur):
    """A few wide patches on the default tiles: the image of smaller tiles bit for bit, in
    at most a quarter more time (tiles of twice the area, half as many workgroups)."""
    side, n = 512, 2621
    rng = np.random.default_rng(blur)
    b = gu.batch_for([(side, side)], [(4, 4)], [n])
    x, y, z, d, I0 = (gu.to_dev(rng.uniform(*r, n).astype(np.float32))
                      for r in ((-5, side + 5), (-5, side + 5), (-1, 1), (4.0, 16.0), (0.01, 0.02)))
    rp = sp.render_params(0.5, 16.0, blur, 0.7, 0.0, 0)
    best, img = {}, {}
    for tile in ((64, 64), (64, 32)):
        tl = sp.tiling(*tile, 2048, 64)
        ws = sp.alloc_workspace(b, rp, tl)
        for _ in range(8):
            sp.timing_read(None)
            sp.timing_enable(True)
            img[tile] = sp.render_pair(b, x, y, y, x, z, d, I0, rp, tl, workspace=ws)
            torch.cuda.synchronize()
            sp.timing_enable(False)
            best[tile] = min(best.get(tile, 1e9), sp.timing_read("render_tile")[0])
    sp.timing_read(None)
    assert torch.equal(img[(64, 64)], img[(64, 32)])
    assert best[(64, 64)] <= 1.25 * best[(64, 32)], best
