"""Bins of tiles with more entries than a block sorts at a time (12 288), whose
rounds several blocks share: a bin at and just above that size, tens of rounds,
a sliver of the depth range that holds most of a bin, single depths, crowded
and other bins side by side in several views, and every bin of a view crowded.
Membership and order are exact against the CPU oracle, and repeated calls give
the same lists (the place of a shared bin's lists is reserved by whichever block
comes first)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _cloud(n, seed, half, z, log_scale=-3.5):
    """n Gaussians in front of an identity camera at depths z, spread over
    +-half of the depth."""
    g = np.random.default_rng(seed)
    sc = W.random_scene(n, seed=seed, log_scale_mu=log_scale, log_scale_sd=0.2)
    sc.mean[:, 2] = np.asarray(z(g, n), np.float32)
    sc.mean[:, :2] = (g.uniform(-half, half, (n, 2)) * sc.mean[:, 2:]).astype(np.float32)
    return sc


def _check(gsr, sc, cams, tiles, capacity=None, largest=None):
    sizes = [(c.width, c.height) for c in cams]
    r = gsr.Renderer()
    r.plan(sc.n, sizes, capacity)
    cfg = gsr.Config()
    g, packed = H.gpu_scene(gsr, sc), gsr.pack_cameras(cams)
    first = None
    for _ in range(3):
        r.render_forward(g, packed, cfg)
        rng, ids = (x.numpy() for x in r.debug_tiles())
        ids = ids[:rng[-1, 1]]
        if first is not None:
            assert np.array_equal(rng, first[0]) and np.array_equal(ids, first[1])
        first = rng.copy(), ids.copy()
    ocfg = H.oracle_cfg_of(cfg)
    off = total = 0
    for v, cam in enumerate(cams):
        proj = O.project(sc, cam, ocfg.as_f32())
        T = proj["TX"] * proj["TY"]
        some = None if tiles is None else tiles(rng[off:off + T])
        H.check_view_lists(rng, ids, off, v * sc.n, proj, O.tile_lists(proj), cam.width, cam.height, ocfg, tiles=some)
        off += T
        total += H.rect_pairs(proj)
    assert r.pair_count() == total
    lengths = rng[:, 1] - rng[:, 0]
    if largest is not None:
        assert lengths.max() >= largest
    return lengths


def _longest(k):
    return lambda rng: np.argsort(rng[:, 0] - rng[:, 1], kind="stable")[:k].tolist()


@pytest.mark.parametrize("n", [12_287, 12_288, 12_289, 24_576, 24_577])
def test_one_tile_at_the_rounds_size(gsr_lib, n):
    gsr = gsr_lib
    print("CASE crowded one tile", n, flush=True)
    sc = _cloud(n, n, 0.1, lambda g, k: g.uniform(1.0, 3.0, k))
    sc.opacity_logit[:] = 3.0
    cam = W.camera_small().with_size(16.0, 16.0, 7.5, 7.5, 16, 16)
    lengths = _check(gsr, sc, [cam], None)
    assert lengths[0] == n


DEPTHS = {
    "spread": lambda g, n: g.uniform(1.0, 4.0, n),
    # most of the bin in a part of the histogram, and one entry far away
    "sliver": lambda g, n: np.where(np.arange(n) == 11, 9000.0, np.where(g.random(n) < 0.8, 2.0 + 1e-4 * g.random(n),
                                                                        g.uniform(1.0, 4.0, n))),
    "flat": lambda g, n: np.full(n, 2.0),
    "two_depths": lambda g, n: np.where(g.random(n) < 0.5, 1.5, 2.5),
    "ties": lambda g, n: np.round(g.uniform(1.0, 4.0, n), 3),
}


@pytest.mark.parametrize("depths", list(DEPTHS))
@pytest.mark.parametrize("n", [40_000, 200_000])
def test_many_rounds(gsr_lib, depths, n):
    gsr = gsr_lib
    print("CASE crowded rounds", depths, n, flush=True)
    sc = _cloud(n, 3, 0.25, DEPTHS[depths])
    cam = W.camera_small().with_size(24.0, 24.0, 15.5, 15.5, 32, 32)
    _check(gsr, sc, [cam], _longest(2), largest=n // 4)


def test_a_map_from_afar(gsr_lib):
    """A corner of 4 x 4-tile bins crowded, the other bins empty or sparse."""
    gsr = gsr_lib
    sc = _cloud(120_000, 6, 0.04, lambda g, n: g.uniform(5.0, 7.0, n), log_scale=-5.0)
    sc.mean[:3000, :2] *= 12.0
    cam = W.camera_tum()
    _check(gsr, sc, [cam], lambda rng: _longest(6)(rng) + [0, 7, 600, 1199], largest=10_000)


def test_crowded_views_beside_others(gsr_lib):
    gsr = gsr_lib
    sc = _cloud(90_000, 7, 0.3, lambda g, n: g.uniform(1.0, 4.0, n))
    cam = W.camera_small()
    cams = [cam.with_size(20.0, 20.0, 15.5, 15.5, 32, 32), cam.with_size(500.0, 500.0, 319.5, 239.5, 640, 480),
            cam.with_size(8.0, 8.0, 47.5, 31.5, 97, 65), cam.with_size(60.0, 60.0, 79.5, 59.5, 160, 120)]
    _check(gsr, sc, cams, lambda rng: _longest(2)(rng) + [1], largest=20_000)


@pytest.mark.parametrize("n", [9_000, 30_000])
def test_single_depths_in_several_views(gsr_lib, n):
    """Bins and rounds of one depth are sorted by index: in views whose record
    ids do not start at 0."""
    gsr = gsr_lib
    sc = _cloud(n, 10, 0.3, lambda g, k: np.full(k, 2.0))
    cam = W.camera_small()
    _check(gsr, sc, [cam.with_size(20.0 + v, 20.0, 15.5, 15.5, 32, 32) for v in range(3)], _longest(1), largest=n // 6)


def test_every_bin_crowded(gsr_lib):
    gsr = gsr_lib
    sc = _cloud(14_000, 8, 0.6, lambda g, n: g.uniform(2.0, 4.0, n), log_scale=0.3)
    sc.opacity_logit[:] = 4.0
    cam = W.camera_small().with_size(120.0, 120.0, 111.5, 79.5, 224, 160)
    lengths = _check(gsr, sc, [cam], lambda rng: [0, 69, 139], capacity=3_000_000)
    assert lengths.min() > 12_288


def test_crowded_bins_cost_in_proportion_to_their_entries(gsr_lib):
    """Four times the Gaussians in the same few bins, seen from afar: the tile
    lists take four times as long where their cost is proportional to the
    entries (sixteen where each round reads the whole bin and the rounds follow
    each other); half as much again leaves room for the rounds' uneven ends."""
    import torch
    gsr = gsr_lib
    times = []
    for n in (400_000, 1_600_000):
        sc = _cloud(n, 9, 0.025, lambda g, k: g.uniform(1.0, 3.0, k), log_scale=-8.0)
        cam = W.camera_small().with_size(640.0, 640.0, 319.5, 239.5, 640, 480)
        r = gsr.Renderer()
        r.plan(sc.n, [(640, 480)])
        g, packed, cfg = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), gsr.Config()
        for k in range(8):
            if k == 3:
                torch.cuda.synchronize()
                r.set_profiling(True)
                r.stage_times()
            r.render_forward(g, packed, cfg)
        t = r.stage_times()
        times.append(t["pair_sort"] / t["calls"])
    print("lists of 400 000, 1 600 000 (ms):", times, flush=True)
    assert times[1] <= 6.0 * times[0]
