"""What calls answer at the limits of a rule: depth spans past a plan's sort,
degenerate and very large Gaussians, equal results however a call is cut up."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _front_view(width, height, focal, n_views=1, turn=0.0):
    """Cameras at the origin that look along +z, rolled by `turn`."""
    import synth
    c, s = np.cos(turn), np.sin(turn)
    P = np.array([[c, -s, 0, 0], [s, c, 0, 0], [0, 0, 1, 0]], float).reshape(1, 12)
    K = np.array([[focal, focal, width / 2, height / 2]], float)
    return synth.Views(np.repeat(P, n_views, 0), np.repeat(K, n_views, 0),
                       np.array([[width, height]] * n_views, dtype=np.int32))


# both forms of the sort (one block for up to 4096 keys), ranges in half tiles and
# (from 129 tiles across) in pixels
@pytest.mark.parametrize("n", [700, 9000])
@pytest.mark.parametrize("width", [96, 2080])
def test_plan_depth_span_with_invisible_gaussians(n, width):
    """A plan sorts a scene's depth keys by their low 24 bits when they span
    less at creation.  Attributes that change in place so that a key lies exactly
    2^24 - 1 past the nearest one tie with the Gaussians off screen, which come
    first by index and have no ranges: the scene's output is 0, the other scene's
    stands, and with the old attributes the first one's is what it was."""
    import synth
    import paper_2607_02721_amd as gs
    rng = np.random.default_rng(n)
    vw = _front_view(width, 48, 60.0, 3)
    mean = np.stack([rng.uniform(-0.5, 0.5, n), rng.uniform(-0.3, 0.3, n), rng.uniform(2.5, 7.0, n)], 1)
    mean[: n // 2, 0] += 1000.0                      # off screen
    mean[-1] = (0.0, 0.0, 2.0)
    d = gs.DeviceScene.from_scene(synth.make_explicit_scene(mean, -3.0, (1.0, 0, 0, 0), 0.5, 1.0))
    other = gs.DeviceScene.from_scene(synth.make_cluster_scene(3000, 41, 1))
    other_views = synth.make_orbit_views(3, 42, 80, 48)
    plan = gs.Plan([d, other], [vw, other_views])
    assert plan.info()["n_sort3_scenes"] == 2
    first, second = [o.clone() for o in plan.run()]
    torch.cuda.synchronize()
    plan.status()
    assert float(first.max()) > 0 and float(second.max()) > 0
    old = float(d.mean[2, -2])
    near = np.float32(2.0).view(np.uint32)
    d.mean[2, -2] = float((near + np.uint32(0xFFFFFF)).view(np.float32))
    out = [o.clone() for o in plan.run()]
    torch.cuda.synchronize()
    with pytest.raises(gs.GsError) as e:
        plan.status()
    assert e.value.status == 5 and "depth keys spanned" in str(e.value)
    assert float(out[0].abs().max()) == 0
    assert torch.equal(out[1], second)
    d.mean[2, -2] = old
    out = plan.run()
    torch.cuda.synchronize()
    assert torch.equal(out[0], first) and torch.equal(out[1], second)
    plan.close()


def test_needles_without_area_are_absent():
    """Gaussians of one dimension, without dilation, seen by a camera rolled by
    45 degrees: the entries of the 2D covariance are equal, so it has no inverse
    and the Gaussian is absent, as in the FP64 oracle; with the default dilation
    every one is there."""
    import synth
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    n = 200
    rng = np.random.default_rng(1)
    mean = np.zeros((n, 3))
    mean[:, 2] = rng.uniform(1.5, 4.0, n)
    scale = np.full((n, 3), -400.0)                 # exp(2 x -400) is 0 in FP64
    scale[:, 0] = rng.uniform(-4.0, 0.0, n)
    sc = synth.make_explicit_scene(mean, scale, (1.0, 0, 0, 0), 0.5, 1.0)
    vw = _front_view(64, 64, 60.0)
    vw.world_to_cam[0, [0, 1, 4, 5]] = np.sqrt(0.5) * np.array([1, -1, 1, 1])
    d = gs.DeviceScene.from_scene(sc)
    s, st = gs.sensitivity(d, vw, stats=True)
    assert st["n_projected"] == n and float(s.max()) > 0
    assert float(np.max(ora.sensitivity(sc, vw, ora.default_params(dilation=0.0))["s"])) == 0
    s, st = gs.sensitivity(d, vw, dilation=0.0, stats=True)
    assert st["n_projected"] == 0 and float(s.max()) == 0


def test_ranges_of_very_large_footprints():
    """Footprints of 4.5 to 9 x 10^15 pixels in radius, where FP64 numbers are 1
    pixel apart, whose edge crosses the view: the tiles they list are those right of
    the edge (at most a pixel or two off by rounding; the edges stand 4 pixels from
    a tile's border)."""
    import synth
    import paper_2607_02721_amd as gs
    rng = np.random.default_rng(2)
    sc = synth.make_explicit_scene([[0.0, 0.0, 2.0]], 0.0, (1.0, 0, 0, 0), 0.5, 1.0)
    d = gs.DeviceScene.from_scene(sc)
    vw = _front_view(1024, 16, 60.0)
    for k in range(48):
        fx = float(rng.uniform(3.0e15, 5.9e15))
        radius = 3.0 * np.sqrt((0.5 * fx) ** 2 + np.float64(np.float32(0.3)))
        tile = int(rng.integers(1, 63))
        vw.intrinsics[0, 0] = fx
        vw.intrinsics[0, 2] = radius + 16 * tile + (4 if k % 2 else 12)
        _, st = gs.sensitivity(d, vw, stats=True)
        assert st["n_entries"] == 64 - tile, (k, fx, tile)


@pytest.mark.parametrize("mode", ["rgbsum", "l2"])
@pytest.mark.parametrize("floor", [1e-12, 1e-2])
@pytest.mark.parametrize("aggregate", ["ray", "image"])
def test_results_do_not_depend_on_the_chunks(mode, floor, aggregate):
    """36 864 regions in one call and 3 072 at a time: per-ray results are maxima
    of shares, per-image ones maxima over the views of exact integer sums, so how
    many views a chunk holds (which the free memory decides) changes no bit, also
    where rays stop early."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(20_000, 43, 1)
    sc.log_scale[:] += np.float32(1.0)
    sc.opacity[:] = np.float32(0.9)
    vw = synth.make_orbit_views(12, 44, 1024, 768)
    d = gs.DeviceScene.from_scene(sc)
    qm = {"rgbsum": gs.QUERY_RGBSUM, "l2": gs.QUERY_L2}[mode]
    kw = dict(query_mode=qm, aggregate={"ray": gs.AGG_RAY, "image": gs.AGG_IMAGE}[aggregate], share_floor=floor)
    every, _ = gs.sensitivity(d, vw, **kw)
    assert float(every.max()) > 0
    for k in (1, 5):
        some, _ = gs.sensitivity(d, vw, max_views_per_chunk=k, **kw)
        assert torch.equal(every, some), k


@pytest.mark.parametrize("kind,n", [("point", 33), ("point", 2049), ("point", 10_000), ("pairs", 6000),
                                    ("lattice", 8000), ("lattice", 27_000)])
def test_knn_of_ties(kind, n):
    """Clouds in which most distances are equal (all means in one place, in two,
    on a shuffled lattice): ties go to the smaller index, bit for bit as by
    comparing every pair."""
    import paper_2607_02721_amd as gs
    from paper_2607_02721_amd import learned
    g = torch.Generator(device="cuda").manual_seed(n)
    if kind == "lattice":
        side = round(n ** (1 / 3))
        m = torch.stack(torch.meshgrid(*[torch.arange(float(side), device="cuda")] * 3, indexing="ij")).reshape(3, -1)
        m = m[:, torch.randperm(n, generator=g, device="cuda")]
    else:
        m = torch.full((3, n), 0.25, device="cuda")
        if kind == "pairs":
            m[0] += torch.randint(0, 2, (n,), generator=g, device="cuda")
    one = lambda *s: torch.ones(*s, device="cuda")  # noqa: E731
    idx, d2 = learned.knn(gs.DeviceScene(m.contiguous(), -one(3, n), one(4, n), one(n), one(1, 3, n), 0))
    rows = torch.randperm(n, generator=g, device="cuda")[:700]
    d = ((m[:, None] - m[:, rows, None]) ** 2).sum(0)       # exact: multiples of 1/16
    key = (d.view(torch.int32).long() << 32) | torch.arange(n, device="cuda")[None]
    key[torch.arange(len(rows), device="cuda"), rows] = torch.iinfo(torch.int64).max
    best = torch.topk(key, 16, dim=1, largest=False).values.sort(1).values
    assert torch.equal(idx[rows], (best & 0xFFFFFFFF).int())
    assert torch.equal(d2[rows], (best >> 32).int().view(torch.float32))


@pytest.mark.parametrize("xcd_remap", [0, 1])
def test_plan_launch_orders_agree(xcd_remap, monkeypatch):
    """A plan of two scenes, 133 200 and 9 360 regions, each a launch of its own
    (no room for compacted lists) and both in one: in tile order (xcd_remap 0) and
    with the longest lists first, the scenes' sensitivities are those of their
    own calls."""
    import synth
    import paper_2607_02721_amd as gs
    batch = [(gs.DeviceScene.from_scene(synth.make_cluster_scene(3000, 47 + k, 1)),
              synth.make_orbit_views(v, 49 + k, 1280, 720)) for k, v in enumerate((37, 3))]
    ref = [gs.sensitivity(d, vw)[0] for d, vw in batch]
    for room in ("0", None):
        if room is None:
            monkeypatch.delenv("GS_COMPACT_POOL_GB")
        else:
            monkeypatch.setenv("GS_COMPACT_POOL_GB", room)
        plan = gs.Plan([d for d, _ in batch], [v for _, v in batch])
        assert plan.info()["n_launches"] == (1 if room is None else 2)
        plan.set_config(0, xcd_remap)
        for _ in range(2):
            outs = plan.run()
        torch.cuda.synchronize()
        for o, r in zip(outs, ref):
            assert float(r.max()) > 0
            assert torch.equal(o, r)
        plan.close()


@pytest.mark.parametrize("n,views,height,chunks", [(60_000, 1, 136, 235), (60_000, 200, 136, 59), (20_000, 4096, 272, 2)])
def test_segment_count(n, views, height, chunks):
    """gs_stats.n_bins: the (tile, chunk) segments of the call, whose chunks hold
    2^8, 2^10 and 2^14 depth positions here."""
    import synth
    import paper_2607_02721_amd as gs
    d = gs.DeviceScene.from_scene(synth.make_cluster_scene(n, 45, 0))
    vw = synth.make_orbit_views(views, 46, 16, height)
    _, st = gs.sensitivity(d, vw, stats=True)
    assert st["n_bins"] == views * (height // 16 + (height % 16 > 0)) * chunks


# 40 000 tile rows: chunks of 2^13 and 2^14 positions, eight and sixteen batches of
# 1024 (half as many of 2048 with a mask), the last chunk of 808 and 616 positions
@pytest.mark.parametrize("n", [9000, 17_000])
@pytest.mark.parametrize("width", [48, 288])
def test_emission_of_long_chunks(n, width):
    """Rows that meet few positions of a batch leave some over for the next, with
    and without a ray mask, with 3 active tiles per row (taken one by one) and 18
    (the general form): the selected rays' objectives equal the unmasked call's, and
    a view's equal those of a call of its own, whose chunks are one batch."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(n, 51, 0)
    sc.log_scale[:] -= np.float32(1.5)
    vw = synth.make_orbit_views(400, 52, width, 800)
    d = gs.DeviceScene.from_scene(sc)
    kw = dict(diag=False, tile=(16, 8))
    whole = gs.render_objective(d, vw, **kw)["per_ray"]
    assert float(whole.max()) > 0
    rays = width * 800
    mask = torch.full(((400 * rays + 31) // 32,), 0x11111111, dtype=torch.int32, device="cuda")   # every fourth ray
    part = gs.render_objective(d, vw, ray_mask=mask, **kw)["per_ray"]
    assert torch.equal(part[::4], whole[::4])
    assert float(part.view(-1, 4)[:, 1:].abs().max()) == 0
    for v in (0, 133, 399):
        one = gs.render_objective(d, vw.subset([v]), **kw)["per_ray"]
        assert torch.equal(one, whole[v * rays:(v + 1) * rays])


@pytest.mark.parametrize("noalloc", [False, True])
def test_sampler_beyond_the_prefixes_in_lds(noalloc):
    """More than 2048 blocks of quanta (4.2 million Gaussians), whose prefixes a
    draw searches in memory: counts, weights and support equal the oracle's."""
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    n = 4_300_001
    rng = np.random.default_rng(53)
    s = rng.uniform(0, 1, n).astype(np.float32)
    s[rng.uniform(size=n) < 0.3] = 0
    s[100_000:110_000] = 0
    ref = ora.sample(s, 50_000, 9)
    counts, w, sup = gs.sample_coreset(torch.as_tensor(s).cuda(), 50_000, 9, noalloc=noalloc)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), ref["counts"])
    assert np.array_equal(w.cpu().numpy().view(np.uint64), ref["weights"].view(np.uint64))
    assert int(sup.item()) == ref["support"]


def test_knn_four_levels():
    """More than 32 x 64^3 means: four levels of nodes."""
    import paper_2607_02721_amd as gs
    from paper_2607_02721_amd import learned
    n = 8_400_001
    g = torch.Generator(device="cuda").manual_seed(54)
    m = torch.rand(3, n, generator=g, device="cuda")
    m[:, ::3] *= 0.1
    one = lambda *s: torch.ones(*s, device="cuda")  # noqa: E731
    idx, d2 = learned.knn(gs.DeviceScene(m, -one(3, n), one(4, n), one(n), one(1, 3, n), 0))
    rows = torch.cat([torch.randint(0, n, (118,), generator=g, device="cuda"), torch.tensor([0, n - 1], device="cuda")])
    for r in rows.split(20):
        e = [m[c][None, :] - m[c][r][:, None] for c in range(3)]
        d = (e[0] * e[0] + e[1] * e[1]) + e[2] * e[2]
        key = (d.view(torch.int32).long() << 32) | torch.arange(n, device="cuda")[None]
        key[torch.arange(len(r), device="cuda"), r] = torch.iinfo(torch.int64).max
        best = torch.topk(key, 16, dim=1, largest=False).values.sort(1).values
        assert torch.equal(idx[r], (best & 0xFFFFFFFF).int())
        assert torch.equal(d2[r], (best >> 32).int().view(torch.float32))
