"""Tile lists at the sizes where the list building changes its way: a bin of
tiles with more entries than one round sorts, depths crowded into a sliver of
the bin's range, runs of equal depths (short ones, long ones, and longer than
a round), several batches of records in one projection block, and a view with
more bins than a block counts at a time.  Membership and order are exact
against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _flat(n, seed, z):
    """n Gaussians in front of an identity camera at camera depths z."""
    sc = W.random_scene(n, seed=seed, xy=0.6, z=(1.0, 2.0), log_scale_mu=-3.5)
    sc.mean[:, 2] = z(np.random.default_rng(seed + 100), n).astype(np.float32)
    return sc


CASES = {
    # one round holds 12 288 entries at most
    "rounds": (44_000, (32, 32), lambda r, n: r.uniform(1.0, 4.0, n)),
    # within a few ulp of two depths, and one far away: one slot for thousands
    "crowded": (6_000, (32, 32), lambda r, n: np.where(np.arange(n) == 7, 900.0, np.where(
        r.random(n) < 0.5, 1.5, 2.5) + r.integers(0, 40, n) * 2.4e-7)),
    "pairs_equal": (4_000, (48, 40), lambda r, n: np.repeat(r.uniform(1.0, 4.0, n // 2), 2)[r.permutation(n)]),
    "all_equal": (3_000, (48, 40), lambda r, n: np.full(n, 2.0)),
    "all_equal_rounds": (40_000, (32, 32), lambda r, n: np.full(n, 2.0)),
    "few": (3, (17, 33), lambda r, n: r.uniform(1.0, 4.0, n)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_lists_of_one_view(gsr_lib, case):
    gsr = gsr_lib
    n, size, z = CASES[case]
    print("CASE lists", case, n, size, flush=True)
    sc = _flat(n, 5, z)
    cam = W.camera_small().with_size(24.0, 24.0, (size[0] - 1) / 2, (size[1] - 1) / 2, *size)
    r = gsr.Renderer()
    r.plan(n, [size])
    cfg = gsr.Config()
    r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    again = tuple(x.numpy() for x in r.debug_tiles())
    assert np.array_equal(rng, again[0]) and np.array_equal(ids[:rng[-1, 1]], again[1][:rng[-1, 1]])
    ocfg = H.oracle_cfg_of(cfg)
    proj = O.project(sc, cam, ocfg.as_f32())
    assert r.pair_count() == H.rect_pairs(proj)
    n_or, n_gpu, _ = H.check_view_lists(rng, ids, 0, 0, proj, O.tile_lists(proj), *size, ocfg)
    assert n_gpu > 0 and (case != "rounds" or (rng[:, 1] - rng[:, 0]).max() > 12_288)


def test_lists_of_batches_and_views(gsr_lib):
    """150 000 records a view in several views: four PRE_BLOCKs of records a
    block, whose survivors of the early test fill one to three batches."""
    gsr = gsr_lib
    sc = W.room_scene(150_000, seed=3)
    cam = W.camera_tum_coarse()
    cams = [cam, W.perturb_pose(cam, [0.1, 0.0, 0.1, 0.0, 0.3, 0.0]), cam.with_size(30.0, 30.0, 47.5, 31.5, 96, 64),
            W.perturb_pose(cam.with_size(60.0, 60.0, 50.0, 33.0, 101, 67), [0.0, 0.2, -0.1, 0.1, -0.8, 0.1])]
    sizes = [(c.width, c.height) for c in cams]
    r = gsr.Renderer()
    r.plan(sc.n, sizes)
    cfg = gsr.Config()
    r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras(cams), cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    ocfg = H.oracle_cfg_of(cfg)
    off = total = 0
    for v, c in enumerate(cams):
        proj = O.project(sc, c, ocfg.as_f32())
        T = proj["TX"] * proj["TY"]
        tiles = np.random.default_rng(v).choice(T, 6, replace=False).tolist()
        H.check_view_lists(rng, ids, off, v * sc.n, proj, O.tile_lists(proj), c.width, c.height, ocfg, tiles=tiles)
        off += T
        total += H.rect_pairs(proj)
    assert r.pair_count() == total


def test_lists_of_a_view_with_many_bins(gsr_lib):
    """68 x 68 bins of 4 x 4 tiles: more than a projection block counts at a
    time, with Gaussians large enough to reach bins of both turns."""
    gsr = gsr_lib
    size = (4340, 4352)
    sc = W.random_scene(900, seed=8, xy=1.3, z=(1.5, 3.0), log_scale_mu=-2.5, log_scale_sd=0.7)
    cam = W.camera_small().with_size(2600.0, 2600.0, 2169.5, 2175.5, *size)
    r = gsr.Renderer()
    r.plan(sc.n, [size], pair_capacity=4_000_000)
    cfg = gsr.Config()
    r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    ocfg = H.oracle_cfg_of(cfg)
    proj = O.project(sc, cam, ocfg.as_f32())
    assert r.pair_count() == H.rect_pairs(proj)
    tiles = np.random.default_rng(1).choice(proj["TX"] * proj["TY"], 150, replace=False).tolist()
    _, n_gpu, _ = H.check_view_lists(rng, ids, 0, 0, proj, O.tile_lists(proj), *size, ocfg, tiles=tiles)
    assert n_gpu > 0


@pytest.mark.parametrize("n", [100, 512, 1500])
def test_lists_of_wide_gaussians(gsr_lib, n):
    """Gaussians about 500 px wide and a few tile rows high: a batch of 512 has
    more entries than the count's list holds (3 072) while all its tile rows
    stay in LDS; 100 fit the list, 1 500 take three batches of the two kinds."""
    gsr = gsr_lib
    size = (640, 480)
    sc = W.needle_scene(n, seed=2, z=(2.5, 3.5), half_width=0.4, sigma_y=(0.2, 0.5), sigma_thin=0.004)
    sc.mean[:, :2] = sc.mean[:, 1::-1]  # lying instead of standing
    sc.mean[:, 0] *= 2.0
    sc.log_scale[:, :2] = sc.log_scale[:, 1::-1]
    cam = W.camera_tum()
    r = gsr.Renderer()
    r.plan(n, [size], pair_capacity=2_000_000)
    cfg = gsr.Config()
    r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    ocfg = H.oracle_cfg_of(cfg)
    proj = O.project(sc, cam, ocfg.as_f32())
    rect = proj["rect"][proj["valid"]]
    rows, bins = rect[:, 3] - rect[:, 2] + 1, (rect[:, 1] // 4 - rect[:, 0] // 4 + 1) * (rect[:, 3] // 4 - rect[:, 2] // 4 + 1)
    assert rows.sum() / n <= 6 and bins.sum() / n > 7  # 512: at most 3 072 rows, more than 3 072 entries
    assert r.pair_count() == H.rect_pairs(proj)
    tiles = np.random.default_rng(n).choice(proj["TX"] * proj["TY"], 80, replace=False).tolist()
    _, n_gpu, _ = H.check_view_lists(rng, ids, 0, 0, proj, O.tile_lists(proj), *size, ocfg, tiles=tiles)
    assert n_gpu > 0


@pytest.mark.parametrize("fill", ["zeros", "ones", "random", "stale", "stale_full", "no_tag"])
def test_lists_in_a_workspace_of_any_contents(gsr_lib, fill):
    """A workspace's first call, whatever its memory held, and a call behind one
    that left the entries' cursor (words 32-33: a tag above a count) above 0:
    the same lists, or the overflow report once when the count leaves no room."""
    import torch
    gsr = gsr_lib
    n, size = 20_000, (96, 64)
    sc, cam = W.random_scene(n, seed=4), W.camera_small().with_size(70.0, 70.0, 47.5, 31.5, *size)
    r = gsr.Renderer()
    r.plan(n, [size], pair_capacity=400_000)
    g, cams, cfg = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), gsr.Config()
    r.render_forward(g, cams, cfg)
    pairs = r.pair_count()
    want = [x.numpy() for x in r.debug_tiles()]
    words = r.workspace.view(torch.int32)
    count = {"stale": 1234, "stale_full": 400_000, "no_tag": -(0xA53C7 << 44)}.get(fill)
    for again in range(3):
        if count is None and again == 0:
            r.workspace.view(torch.uint8).copy_({
                "zeros": torch.zeros_like, "ones": lambda t: torch.full_like(t, 255),
                "random": lambda t: torch.randint(0, 256, t.shape, dtype=torch.uint8, device=t.device)}[fill](
                    r.workspace.view(torch.uint8)))
        elif count is not None and again == 0:
            cursor = (0xA53C7 << 44) + count
            words[32] = cursor & 0x7FFFFFFF
            words[33] = (cursor >> 32) - 2**32 if cursor >> 63 else cursor >> 32
        r.render_forward(g, cams, cfg, check=False)
        torch.cuda.synchronize()
        if fill in ("stale_full", "no_tag") and again == 0:
            with pytest.raises(gsr.GsrError):
                r.check_overflow()
            continue
        r.check_overflow()
        assert r.pair_count() == pairs
        got = [x.numpy() for x in r.debug_tiles()]
        assert np.array_equal(got[0], want[0])
        assert np.array_equal(got[1][:want[0][-1, 1]], want[1][:want[0][-1, 1]])


def test_no_entries_in_a_workspace_never_used(gsr_lib):
    """Nothing in view and garbage in the header: no overflow, empty lists."""
    import torch
    gsr = gsr_lib
    sc, cam = W.random_scene(500, seed=4), W.camera_small()
    sc.mean[:, 2] -= 50.0
    r = gsr.Renderer()
    r.plan(500, [(cam.width, cam.height)])
    r.workspace.view(torch.uint8).fill_(255)
    out = r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), gsr.Config())
    assert r.pair_count() == 0 and float(out["T_final"].min()) == 1.0
