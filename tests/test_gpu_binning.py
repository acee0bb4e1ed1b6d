"""Key lists of the binning's variants at the sizes where one takes over from another, bit-exact
against the oracle: items sorted by rank (up to 8,192 Gaussians) or by radix passes, whose scatter sums
the digit counts itself (up to 32 blocks of 4,096 items per view) or has them scanned; pairs sorted
by one pass over the tile id (9 to 11 bits) or by several; views whose items are partly or all culled."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2410_20686_amd import scenes
from tests import _gpu as G
from tests._util import settings

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    """Small footprints, an eighth of the Gaussians sharing positions (equal depths) with others."""
    sc = scenes.sphere_scene(n, 0, seed=seed)
    sc.scales *= np.float32(0.05)
    twin = np.arange(n - n // 8, n)
    sc.means[:, twin] = sc.means[:, twin - n // 2]
    return sc


def _check(sc, cams, st, capacity=None):
    res = G.run_gpu(sc, cams, st, pair_capacity=capacity, return_rast=True)
    keys, gauss = res["rast"].keys()
    okeys, ovals = O.keys(sc, cams, st)
    assert res["status"]["n_pairs"] == len(okeys)
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), okeys)
    np.testing.assert_array_equal(gauss.cpu().numpy().astype(np.uint32), ovals)
    return res


@pytest.mark.parametrize("n", [1, 255, 256, 257, 2048, 2049, 8192, 8193, 131072, 131073])
@pytest.mark.parametrize("views", [1, 3])
def test_item_sort(n, views):
    """Three views: the middle one is too far away to keep anything."""
    cams = scenes.yaw_cameras(views, 64, 32, seed=n)
    if views == 3:
        cams.cams[1, 9:] += np.float32(2e4)
    _check(_scene(n, seed=n), cams, settings())


@pytest.mark.parametrize("n", [3000, 20000])
def test_items_of_partial_views(n):
    """Six faces of a cubemap, each keeping a part of the Gaussians, next to a panorama."""
    faces, erp = scenes.cubemap_cameras(64), scenes.yaw_cameras(1, 128, 64, seed=n)
    cams = scenes.Cameras(np.concatenate([faces.cams, erp.cams]), np.concatenate([faces.wh, erp.wh]))
    _check(_scene(n, seed=n), cams, settings(pinhole={v: (32.0, 32.0, 32.0, 32.0) for v in range(6)}))


@pytest.mark.parametrize("wh,capacity", [((128, 128), None), ((136, 128), None), ((512, 256), None), ((520, 256), None),
                                         ((512, 256), 1024 * 4096), ((512, 256), 1024 * 4096 + 1), ((1024, 512), None),
                                         ((1032, 512), None)])
def test_tile_sort(wh, capacity):
    """256 tiles of 8x8 (one pass of a byte), 272 and 2,048 (one wide pass), 2,080 (two passes); 2,048
    with the most sort blocks of the wide pass and one more; 8,192 and 8,256 (the queue's one-workgroup
    limit)."""
    sc = _scene(9001, seed=5)
    cams = scenes.yaw_cameras(1, *wh, seed=5)
    res = _check(sc, cams, settings(tile=8), capacity)
    rast, tiles = res["rast"], wh[0] * wh[1] // 64
    import torch
    p = rast.plan
    q = rast.ws[p.off_queue + 64:p.off_queue + 64 + 4 * tiles].view(torch.int32).cpu().numpy()
    r = rast.ws[p.off_ranges:p.off_ranges + 8 * tiles].view(torch.int32).cpu().numpy().reshape(tiles, 2)
    assert np.array_equal(np.sort(q), np.arange(tiles))
    length = (r[:, 1] - r[:, 0])[q]
    assert length.sum() == res["status"]["n_pairs"] and length.min() >= 0
    # longest first, within the 1/32 octave of a cost bucket
    assert np.all(length[1:] <= length[:-1] * 2.0 ** (1 / 16) + 1)
