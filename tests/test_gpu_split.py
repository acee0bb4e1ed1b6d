"""Lists split into quadrant tasks at tiles of 16x16: which lists the queue splits, and the quadrant
compositors at list lengths around the entries they take together (4 forward, 2 reverse), their
groups of seven and their batches of 64.  Whole-tile compositing in tile id order is the reference:
images and depths bit-identical; the compositor's 2D gradients, whose per-(entry, tile) float sums run
over other pixels, to the parity tolerance."""
import numpy as np
import pytest

from paper_2410_20686_amd import scenes
from tests import _gpu as G
from tests._util import settings

pytestmark = pytest.mark.gpu


def _bucket(x):
    x = np.asarray(x, dtype=np.int64)
    b = 1 + ((x.astype(np.float32).view(np.uint32).astype(np.int64) - 0x3F800000) >> 18)
    return np.where(x == 0, 0, b)


def _expected_split(lengths):
    """Lists of at least 1/4096 of all pairs, or the 128 longest of at least half that and 1024 pairs,
    and of at least 64 pairs from 4096 tiles on; at most max(1024, tiles / 8)."""
    tiles, pairs = len(lengths), int(lengths.sum())
    b = _bucket(lengths)
    floor = 64 if tiles >= 4096 else 1
    long = int((b >= _bucket(max(floor, pairs // 4096))).sum())
    top = min(int((b >= _bucket(max(1024, pairs // 8192))).sum()), 128)
    return min(max(long, top), tiles if tiles < 1024 else max(1024, tiles // 8))


def _run(sc, cams, st, dL):
    import torch
    res = G.run_gpu(sc, cams, st, dL=dL, return_rast=True, split_bwd=True)
    rast = res["rast"]
    p = rast.plan
    tiles = int(p.tile_base[cams.n_views])
    r = rast.ws[p.off_ranges:p.off_ranges + 8 * tiles].view(torch.int32).cpu().numpy().reshape(tiles, 2)
    res["lengths"] = (r[:, 1] - r[:, 0]).astype(np.int64)
    res["header"] = rast.ws[p.off_queue:p.off_queue + 64].view(torch.int32).cpu().numpy()
    depth = torch.empty(rast.pixels, dtype=torch.float32, device="cuda")
    rgb, _ = rast.render_fwd(out_depth=depth)
    np.testing.assert_array_equal(rgb.cpu().numpy(), res["rgb"])
    res["depth"] = depth.cpu().numpy()
    return res


def _check(sc, cams, st, schedules=("queue",)):
    dL = scenes.upstream_gradient(cams, seed=7)
    base = _run(sc, cams, dict(st, schedule="tile_id"), dL)
    assert base["header"][7] == 0
    for s in schedules:
        res = _run(sc, cams, dict(st, schedule=s), dL)
        split = _expected_split(res["lengths"])
        assert res["header"][6] == split and res["header"][7] == split
        for k in ("rgb", "T", "depth"):
            np.testing.assert_array_equal(res[k], base[k])
        G.assert_grads_close(res, base, names=("g2d",))
    return split, base["lengths"]


@pytest.mark.parametrize("opacity", [0.02, 0.999])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 65, 129, 258])
def test_quadrant_list_lengths(n, opacity):
    """A stack of n footprints across the image's left and right border; nearly opaque ones reach the
    alpha clamp and stop pixels inside a run."""
    sc = scenes.sphere_scene(n, 1, seed=n)
    dist = np.linspace(1.0, 3.0, n)
    sc.means[:] = np.stack([0.02 * dist, 0.1 * dist, -dist])
    sc.scales[:] = (0.15 * dist)[None]
    sc.opacities[:] = np.float32(opacity)
    split, lengths = _check(sc, scenes.identity_cameras(64, 32), settings(tile=16))
    assert split > 0 and lengths.max() == n


@pytest.mark.parametrize("n,scale,crowd,top", [(3000, 0.6, 0.03, False), (6000, 10.0, 0.6, True)])
def test_split_rule(n, scale, crowd, top):
    """8,192 tiles: few pairs (the lists of 64 and more are split), and 4 million of them and more
    (lists below 1/4096 of the pairs are split up to the 128th)."""
    sc = scenes.sphere_scene(n, 0, seed=5)
    sc.means[:, : n // 4] = sc.means[:, :1] + np.float32(crowd) * sc.means[:, : n // 4]  # one direction
    sc.scales *= np.float32(scale)
    sc.opacities *= np.float32(0.05)
    split, lengths = _check(sc, scenes.identity_cameras(2048, 1024), settings(tile=16), ("queue", "persistent"))
    assert 0 < split < len(lengths)
    assert (split == 128) == top


@pytest.mark.parametrize("batch", [64, 128, 256])
@pytest.mark.parametrize("n,opacity", [(1100, 0.02), (1301, 0.6)])
def test_long_lists_of_32_pixel_tiles(n, opacity, batch):
    """Forward in sixteen tasks per 32x32 tile from 1,024 pairs on, the reverse in four with the masks put
    together: nothing but the order of the FP64 totals may differ from the launch without a queue.  Faint
    footprints keep every pixel to the end of its list; others stop quadrants at different entries."""
    sc = scenes.sphere_scene(n, 0, seed=n)
    dist = np.linspace(1.0, 3.0, n)
    sc.means[:] = np.stack([0.02 * dist, 0.1 * dist, -dist]) + 0.1 * np.random.default_rng(n).standard_normal((3, n))
    sc.scales[:] = np.abs(sc.scales) * np.float32(3.0)
    sc.opacities[:] = np.float32(opacity)
    cams = scenes.identity_cameras(256, 128)
    st = settings(tile=32, batch=batch, batch_bwd=batch)
    dL = scenes.upstream_gradient(cams, seed=7)
    base = _run(sc, cams, dict(st, schedule="tile_id"), dL)
    assert base["header"][9] == 0
    fine = int((_bucket(base["lengths"]) >= _bucket(1024)).sum())
    assert 0 < fine < len(base["lengths"])
    for s in ("queue", "persistent"):
        res = _run(sc, cams, dict(st, schedule=s), dL)
        assert res["header"][8] == fine and res["header"][9] == fine
        for k in ("rgb", "T", "depth"):
            np.testing.assert_array_equal(res[k], base[k])
        G.assert_grads_close(res, base, names=("g2d",), rtol=1e-6, floor=1e-9)


@pytest.mark.parametrize("schedule", ["queue", "tile_id"])
def test_entry_that_only_stops_pixels_gets_no_gradient(schedule):
    """The third of three footprints on one pixel reaches only that pixel, which stops at it; a fourth lies
    behind.  The upstream gradient is NaN elsewhere in the 8x8 block: none of it may reach the third, which
    contributes to no pixel."""
    from tests.test_gpu_reverse_step import H, W, _g2d, _scene
    sc = _scene([66.5, 66.5, 66.5, 70.5], [34.5, 34.5, 34.5, 36.5], [0.999, 0.98997, 0.008, 0.5], 1e-3,
                radius=np.array([2.0, 2.2, 2.4, 2.6]))
    dL = np.random.default_rng(4).standard_normal((3, H, W)).astype(np.float32)
    dL[:, 38, 65] = np.nan
    T = G.run_gpu(sc, scenes.identity_cameras(W, H), settings(tile=16, schedule=schedule))["T"].reshape(H, W)
    assert 1e-4 <= T[34, 66] < 1.008e-4 and T[38, 65] == 1.0
    g, _ = _g2d(sc, settings(tile=16, schedule=schedule), dL.ravel())
    assert (g[2] == 0.0).all()
    assert (g[[0, 1, 3]][:, 5] != 0.0).all()


@pytest.mark.parametrize("schedule", ["queue", "tile_id"])
def test_infinite_colour_that_reaches_no_pixel(schedule):
    """Faint footprints between the pixel centres of an 8x8 block, among others that cover it: they are in
    its list but reach no pixel, so the image is that of the others, whatever their colours (here past the
    float range)."""
    n, m = 6, 32
    u, v = np.r_[np.full(n, 67.3), np.full(m, 68.0)], np.r_[np.full(n, 35.6), np.full(m, 36.0)]
    from tests.test_gpu_reverse_step import H, W, _scene
    sc = _scene(u, v, np.r_[np.full(n, 0.3), np.full(m, 0.0045)], np.r_[np.full(n, 0.2), np.full(m, 1e-3)][:, None],
                radius=np.r_[np.linspace(2.0, 3.0, n), np.linspace(1.9, 3.1, m)])
    rng = np.random.default_rng(12)
    sh = 0.3 * rng.standard_normal((48, n + m)).astype(np.float32)
    sh[:, n:] = np.float32(3e38) * rng.choice([-1.0, 1.0], (48, m))
    sc = scenes.Scene(sc.means, sc.scales, sc.quats, sc.opacities, sh, 3)
    cams, st = scenes.identity_cameras(W, H), settings(tile=16, schedule=schedule)
    res = G.run_gpu(sc, cams, st, return_rast=True)
    colour = res["rast"].records()[n:, 8:11].cpu().numpy()
    assert np.isinf(colour).any()
    only = G.run_gpu(sc.subset(np.arange(n)), cams, st)
    np.testing.assert_array_equal(res["rgb"], only["rgb"])
    np.testing.assert_array_equal(res["T"], only["T"])
    assert only["T"].reshape(H, W)[36, 68] < 0.9


@pytest.mark.parametrize("batch,batch_bwd", [(64, 64), (64, 128), (256, 64)])
@pytest.mark.parametrize("opacity", [0.02, 0.6])
def test_more_long_lists_than_sixteen_task_tiles(opacity, batch, batch_bwd):
    """Four views of 512x256 at 32x32 tiles whose 512 lists are nearly all long: the first 256 of the queue
    take sixteen tasks each, the others four, forward and reverse staging batches of their own."""
    sc = scenes.sphere_scene(1301, 0, seed=21)
    sc.scales[:] = np.float32(2.0) * np.linalg.norm(sc.means, axis=0)[None] * np.linspace(0.2, 2.0, 1301)
    sc.opacities[:] = np.float32(opacity)
    cams = scenes.yaw_cameras(4, 512, 256, seed=21)
    st = settings(tile=32, batch=batch, batch_bwd=batch_bwd)
    dL = scenes.upstream_gradient(cams, seed=7)
    base = _run(sc, cams, dict(st, schedule="tile_id"), dL)
    assert len(base["lengths"]) == 512 and base["header"][9] == 0
    fine = int((_bucket(base["lengths"]) >= _bucket(1024)).sum())
    assert 256 < fine
    for s in ("queue", "persistent"):
        res = _run(sc, cams, dict(st, schedule=s), dL)
        assert res["header"][8] == fine and res["header"][9] == 256
        for k in ("rgb", "T", "depth"):
            np.testing.assert_array_equal(res[k], base[k])
        G.assert_grads_close(res, base, names=("g2d",), rtol=1e-6, floor=1e-9)
