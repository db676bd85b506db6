"""Kernels at the edges of their blocks and at the sizes where a dispatch rule
changes the path, against plain torch in FP64 or against the general path."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 17, 255, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_feature_stats_block_edges(n, offset):
    """Column means and 1/std around the 1024-row blocks, also for a matrix
    that starts 4 or 12 bytes past a 16-byte boundary.  FP64 sums rounded once
    to float32: 2^-24 of the value, and the variance's cancellation (its
    relative error is at most 64 n 2^-53 (mean^2 + var) / var, below 1e-9 for
    these columns)."""
    from paper_2607_02721_amd import learned
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(n * 64 + 4, generator=g, device="cuda") * 2.0 + 1.0
    feat = buf[offset:offset + n * 64].view(n, 64)
    feat[:, 5] = 0.25       # a constant column: 1/std reads 1
    norm = learned.feature_stats(feat).double()
    x = feat.double()
    mean, std = x.mean(0), x.std(0, unbiased=False)
    inv = torch.where(std > 1e-9, 1 / std.clamp_min(1e-30), torch.ones_like(std))
    assert torch.all((norm[0] - mean).abs() <= 2.0 ** -24 * mean.abs() + 1e-12)
    assert torch.all((norm[1] - inv).abs() <= 1.0e-7 * inv)


def _scene(gs, mean):
    n = mean.shape[1]
    one = lambda *s: torch.ones(*s, device="cuda")  # noqa: E731
    return gs.DeviceScene(mean.contiguous(), -3.0 * one(3, n), one(4, n), 0.5 * one(n), 0.1 * one(1, 3, n), 0)


def _brute_knn(mean, k=16):
    """The k nearest other points by float32 (dx dx + dy dy) + dz dz, ties by
    index; a NaN distance is no neighbour."""
    x = mean.T.contiguous()
    n = x.shape[0]
    none = torch.iinfo(torch.int64).max
    idx = torch.full((n, k), -1, dtype=torch.int32, device="cuda")
    d2 = torch.full((n, k), float("inf"), device="cuda")
    for i in range(0, n, 2048):
        r = x[i:i + 2048]
        e = [x[None, :, c] - r[:, None, c] for c in range(3)]
        d = (e[0] * e[0] + e[1] * e[1]) + e[2] * e[2]
        key = (d.view(torch.int32).long() << 32) | torch.arange(n, device="cuda")[None]
        key[torch.isnan(d)] = none
        key[torch.arange(r.shape[0]), torch.arange(i, i + r.shape[0])] = none
        best = torch.sort(key, 1).values[:, :k]
        m = best.shape[1]
        there = best != none
        idx[i:i + 2048, :m] = torch.where(there, (best & 0xFFFFFFFF).int(), torch.full_like(best, -1).int())
        d2[i:i + 2048, :m] = torch.where(there, (best >> 32).int().view(torch.float32), torch.tensor(float("inf")).cuda())
    return idx, d2


@pytest.mark.parametrize("kind", ["normal", "lattice", "line", "copies", "far", "nonfinite"])
@pytest.mark.parametrize("n", [1, 2, 16, 17, 31, 33, 64, 65, 2047, 2049, 4097, 20_000])
def test_knn_tree_edges(kind, n):
    """Neighbour sets and squared distances, bit for bit, around the tree's
    leaves (32 points), waves (64) and nodes (2048 points; a third level from
    131 073 on is test_knn_three_levels), for ties, a flat cloud, coincident
    points, far outliers and non-finite means."""
    import paper_2607_02721_amd as gs
    from paper_2607_02721_amd import learned
    g = torch.Generator(device="cuda").manual_seed(n)
    m = torch.randn(3, n, generator=g, device="cuda")
    if kind == "lattice":
        m = (m * 4).round() / 8
    elif kind == "line":
        m[1:] = 0.25
    elif kind == "copies":
        m = m[:, torch.randint(0, max(1, n // 20), (n,), generator=g, device="cuda")]
    elif kind == "far":
        m[:, :3] *= 1e6
    elif kind == "nonfinite":
        m[0, n // 2] = float("nan")
        m[1, n // 3] = float("inf")
        m[2, n // 5] = -float("inf")
    idx, d2 = learned.knn(_scene(gs, m))
    ri, rd = _brute_knn(m)
    assert torch.equal(idx, ri)
    assert torch.equal(d2, rd)


def test_knn_three_levels():
    import paper_2607_02721_amd as gs
    from paper_2607_02721_amd import learned
    g = torch.Generator(device="cuda").manual_seed(3)
    n = 140_000
    m = torch.randn(3, n, generator=g, device="cuda")
    m[:, ::2] *= 0.02       # half of the cloud in a dense core
    idx, d2 = learned.knn(_scene(gs, m))
    rows = torch.randint(0, n, (500,), generator=g, device="cuda")
    e = [m[c][None, :] - m[c][rows][:, None] for c in range(3)]
    d = (e[0] * e[0] + e[1] * e[1]) + e[2] * e[2]
    key = (d.view(torch.int32).long() << 32) | torch.arange(n, device="cuda")[None]
    key[torch.arange(500), rows] = torch.iinfo(torch.int64).max
    best = torch.topk(key, 16, dim=1, largest=False).values.sort(1).values
    assert torch.equal(idx[rows], (best & 0xFFFFFFFF).int())
    assert torch.equal(d2[rows], (best >> 32).int().view(torch.float32))


@pytest.mark.parametrize("views", [1, 7, 8, 9, 13])
def test_depth_sort_segment_counts(views):
    """Sensitivities of a call whose views fill whole groups of eight sort
    segments, leave some over, or both, against one view per chunk."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(10_000, 5, 1)     # three sort blocks per view
    vw = synth.make_orbit_views(views, 6, 200, 136)
    d = gs.DeviceScene.from_scene(sc)
    one, _ = gs.sensitivity(d, vw)
    two, _ = gs.sensitivity(d, vw, max_views_per_chunk=1)
    assert float(one.max()) > 0
    assert torch.equal(one, two)


@pytest.mark.parametrize("n", [255, 257, 1023, 1025, 30_000, 60_000])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (8, 8)])
def test_binning_chunk_lengths(n, tile):
    """The binning chunk follows the waves a call has: 200 views in one call
    take longer chunks than single views (2^11 against 2^8 positions at
    60 000 Gaussians and 8-pixel rows).  The lists, and so the sensitivities,
    do not depend on it: one call of all views is the maximum of their own."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(n, 8, 0)
    vw = synth.make_orbit_views(200, 9, 64, 136)
    d = gs.DeviceScene.from_scene(sc)
    every, _ = gs.sensitivity(d, vw, tile=tile)
    each = torch.zeros_like(every)
    for v in range(200):
        each = torch.maximum(each, gs.sensitivity(d, vw.subset([v]), tile=tile)[0])
    assert float(every.max()) > 0
    assert torch.equal(every, each)


@pytest.mark.parametrize("aggregate", ["ray", "tile", "image"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (32, 16)])
def test_tile_order_matches_tile_by_tile(aggregate, tile):
    """A call of more than 8 192 regions composites its tiles longest list
    first, one of fewer in tile order; the sensitivities are the same: 41 views
    in one call against each view by itself (the tile count is no multiple of
    the runs the order is dealt in)."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(20_000, 10, 1)
    vw = synth.make_orbit_views(41, 11, 330, 207)
    d = gs.DeviceScene.from_scene(sc)
    agg = {"ray": gs.AGG_RAY, "tile": gs.AGG_TILE, "image": gs.AGG_IMAGE}[aggregate]
    every, _ = gs.sensitivity(d, vw, tile=tile, aggregate=agg)
    each = torch.zeros_like(every)
    for v in range(41):
        each = torch.maximum(each, gs.sensitivity(d, vw.subset([v]), tile=tile, aggregate=agg)[0])
    assert float(every.max()) > 0
    assert torch.equal(every, each)


@pytest.mark.parametrize("mode", ["rgbsum", "nocolor", "l2", "channel"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (8, 16)])
def test_quadrant_and_region_forms_agree(mode, tile):
    """Small calls composite one wave per quadrant, except counting calls, which
    run by regions: the same bits."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(20_000, 12, 2)
    vw = synth.make_orbit_views(3, 13, 333, 205)
    d = gs.DeviceScene.from_scene(sc)
    qm = {"rgbsum": gs.QUERY_RGBSUM, "nocolor": gs.QUERY_NOCOLOR, "l2": gs.QUERY_L2, "channel": gs.QUERY_CHANNEL}[mode]
    quads, _ = gs.sensitivity(d, vw, query_mode=qm, tile=tile)
    regions, st = gs.sensitivity(d, vw, query_mode=qm, tile=tile, stats=True, count_pairs=True)
    assert st["n_live_pairs"] > 0 and float(quads.max()) > 0
    assert torch.equal(quads, regions)


@pytest.mark.parametrize("mode", ["rgbsum", "l2"])
def test_aggregates_by_regions_and_by_quadrants(mode):
    """42 640 regions in one call composite by regions, a view at a time by
    quadrants.  Per-image results are the maximum over the views, bit for bit;
    the per-scene result is a sum of exact integers of each launch, whose unit
    (2^-60 of the launch's A) and division are all that differ."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(20_000, 14, 1)
    vw = synth.make_orbit_views(41, 15, 640, 414)
    d = gs.DeviceScene.from_scene(sc)
    qm = {"rgbsum": gs.QUERY_RGBSUM, "l2": gs.QUERY_L2}[mode]
    every, _ = gs.sensitivity(d, vw, query_mode=qm, aggregate=gs.AGG_IMAGE)
    each, _ = gs.sensitivity(d, vw, query_mode=qm, aggregate=gs.AGG_IMAGE, max_views_per_chunk=1)
    assert float(every.max()) > 0
    assert torch.equal(every, each)
    every, _ = gs.sensitivity(d, vw, query_mode=qm, aggregate=gs.AGG_SCENE)
    each, _ = gs.sensitivity(d, vw, query_mode=qm, aggregate=gs.AGG_SCENE, max_views_per_chunk=1)
    # (float32 sums of up to 64 shares per quadrant, against A in float32)
    assert torch.all((every - each).abs() <= 2e-6 * each + 1e-15)


@pytest.mark.parametrize("log_scale", [-20.0, -6.0, 0.0, 8.0, 30.0])
def test_projection_scale_range(log_scale):
    """Gaussians from far below a pixel (the dilation alone) to scales whose
    conic products leave the range of the shared reciprocal, at the parity bar
    of 1e-5 against the FP64 oracle on the rays neither side calls ambiguous."""
    import synth
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    sc = synth.make_cluster_scene(400, 16, 3)
    sc.log_scale[:, ::2] = np.float32(log_scale)
    sc.opacity[::2] *= np.float32(0.2)
    vw = synth.make_orbit_views(3, 17, 97, 61)
    ref = ora.sensitivity(sc, vw)
    mask_np = synth.pack_bits(~ref["flag"])
    ref = ora.sensitivity(sc, vw, None, mask_np)
    mask = torch.as_tensor(mask_np.view(np.int32)).cuda()
    s, st = gs.sensitivity(gs.DeviceScene.from_scene(sc), vw, ray_mask=mask, stats=True)
    assert st["n_projected"] > 0
    err = np.abs(s.cpu().numpy().astype(np.float64) - ref["s"]) - (1e-5 * ref["s"] + 1e-12)
    assert err.max() <= 0


@pytest.mark.parametrize("per_row", [1, 15, 16, 17, 40, 80])
def test_masked_emission_tiles_per_row(per_row):
    """Ray masks with few active tiles per tile row (emitted tile by tile, up to
    16) and with more (the general form): the selected rays' objectives equal the
    unmasked render's bit for bit, the others read 0."""
    import synth
    import paper_2607_02721_amd as gs
    W, H = 1280, 96
    sc = synth.make_cluster_scene(30_000, 18, 1)
    vw = synth.make_orbit_views(2, 19, W, H)
    rng = np.random.default_rng(per_row)
    keep = np.zeros((2, H, W), bool)
    for v in range(2):
        for ty in range(H // 16):
            for tx in rng.choice(W // 16, per_row, replace=False):
                y, x = 16 * ty + 8 * rng.integers(2), 16 * tx + 8 * rng.integers(2)
                keep[v, y:y + 8, x:x + 8] = True
    mask = torch.as_tensor(synth.pack_bits(keep.reshape(-1)).view(np.int32)).cuda()
    d = gs.DeviceScene.from_scene(sc)
    whole = gs.render_objective(d, vw, diag=False)["per_ray"]
    part = gs.render_objective(d, vw, ray_mask=mask, diag=False)["per_ray"]
    on = torch.as_tensor(keep.reshape(-1)).cuda()
    assert float(whole[on].max()) > 0
    assert torch.equal(part[on], whole[on])
    assert float(part[~on].abs().max()) == 0


@pytest.mark.parametrize("tile", [(8, 8), (32, 32), (8, 32), (32, 8)])
@pytest.mark.parametrize("size", [(65, 63), (31, 33), (1, 1)])
def test_tile_activity_from_single_rays(tile, size):
    """Single selected pixels at any bit of a mask word, first and last pixels
    included: each one's tile is active, so its objective equals the unmasked
    render's bit for bit, and the others read 0."""
    import synth
    import paper_2607_02721_amd as gs
    W, H = size
    sc = synth.make_cluster_scene(3000, 20, 1)
    vw = synth.make_orbit_views(3, 21, W, H)
    rng = np.random.default_rng(W)
    keep = np.zeros((3, H, W), bool)
    keep[rng.integers(0, 3, 9), rng.integers(0, H, 9), rng.integers(0, W, 9)] = True
    keep[0, 0, 0] = keep[2, H - 1, W - 1] = True
    mask = torch.as_tensor(synth.pack_bits(keep.reshape(-1)).view(np.int32)).cuda()
    d = gs.DeviceScene.from_scene(sc)
    whole = gs.render_objective(d, vw, diag=False, tile=tile)["per_ray"]
    part = gs.render_objective(d, vw, ray_mask=mask, diag=False, tile=tile)["per_ray"]
    on = torch.as_tensor(keep.reshape(-1)).cuda()
    assert float(whole.max()) > 0
    assert torch.equal(part[on], whole[on])
    assert float(part[~on].abs().sum()) == 0


@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1025, 5000])
def test_masked_key_runs(n):
    """Kept keys move in runs of 64 by waves of four runs: one selected block
    keeps few Gaussians, at counts around the run and block lengths."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(n, 22, 1)
    vw = synth.make_orbit_views(3, 23, 160, 96)
    keep = np.zeros((3, 96, 160), bool)
    keep[:, 32:64, 48:112] = True
    mask = torch.as_tensor(synth.pack_bits(keep.reshape(-1)).view(np.int32)).cuda()
    d = gs.DeviceScene.from_scene(sc)
    whole = gs.render_objective(d, vw, diag=False)["per_ray"]
    part = gs.render_objective(d, vw, ray_mask=mask, diag=False)["per_ray"]
    on = torch.as_tensor(keep.reshape(-1)).cuda()
    assert float(whole[on].max()) > 0
    assert torch.equal(part[on], whole[on])


def _mlp_case(n, seed):
    from paper_2607_02721_amd import learned
    rng = np.random.default_rng(seed)
    feat = torch.as_tensor(rng.normal(size=(n, 64)).astype(np.float32)).cuda()
    target = torch.as_tensor(rng.normal(size=n).astype(np.float32)).cuda()
    prop = learned.Proposal(seed=seed)
    prop.set_norm(learned.feature_stats(feat) if n > 1 else torch.stack(
        [torch.zeros(64), torch.ones(64)]).reshape(-1).cuda())
    return learned, prop, feat, target


def _mlp_bf16(params, x, target):
    """Network, loss and gradient with the roundings of the BF16 step (weights,
    activations and dZ to BF16), everything else in FP64."""
    def r(t):
        return t.to(torch.float32).to(torch.bfloat16).double()
    P = params.double().cpu()
    W, off = [], 0
    for o, i in ((256, 64), (256, 256), (256, 256), (1, 256)):
        W.append((r(P[off:off + o * i].reshape(o, i)), P[off + o * i:off + o * i + o]))
        off += o * i + o
    h, zs, hs = r(x), [], [r(x)]
    for w, b in W[:3]:
        z = h @ w.T + b
        zs.append(z)
        h = r(z * torch.sigmoid(z))
        hs.append(h)
    out = h @ W[3][0].T + W[3][1]
    e = out[:, 0] - target.double().cpu()
    n = len(e)
    dy = 2 * e / n

    def dsilu(z):
        s = torch.sigmoid(z)
        return s * (1 + z * (1 - s))
    g4 = torch.cat([dy @ hs[3], dy.sum()[None]])
    dz = r(dy[:, None] * W[3][0] * dsilu(zs[2]))
    grads = []
    for k in (2, 1, 0):
        grads.insert(0, torch.cat([(dz.T @ hs[k]).reshape(-1), dz.sum(0)]))
        if k:
            dz = r((dz @ W[k][0]) * dsilu(zs[k - 1]))
    return out[:, 0], (e * e).sum() / n, torch.cat(grads + [g4])


# n: one row, the 64-row block of training and the 128-row block of inference
# and their neighbours, two ranges of the weight gradients with a short last one,
# more blocks than inference has in flight (33 000).
@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 129, 1025, 1663, 33_000])
def test_fused_network_row_counts(n):
    """Prediction, loss and gradient at the edges of the row blocks.  FP32
    accumulation leaves about 1e-6; that moves a value across a rounding
    boundary of BF16, 2^-8 apart, with a probability of 2e-6 / 2^-8 = 5e-4, and
    the value is then 2^-8 off: 2^-8 sqrt(5e-4) = 9e-5 of a layer's norm, six
    layers 2.2e-4.  A single row has few values to average over: 1e-3; the loss
    goes as the square of differences of the size of the outputs: 4e-3."""
    learned, prop, feat, target = _mlp_case(n, 3)
    norm = prop.norm.reshape(2, 64)
    x = ((feat - norm[0]) * norm[1]).cpu()
    want_y, want_loss, want_g = _mlp_bf16(prop.params, x, target)
    y = prop.predict(feat).double().cpu()
    loss, g = prop.gradient(feat, target)
    assert float((y - want_y).norm() / want_y.norm()) <= 1e-3
    assert abs(float(loss) - float(want_loss)) <= 4e-3 * float(want_loss)
    assert float((g.double().cpu() - want_g).norm() / want_g.norm()) <= 1e-3
    # one Adam step with the gradient returned equals the gradient call's
    p0, g2 = prop.params.clone(), torch.empty_like(g)
    loss2 = prop.train_step(feat, target, lr=1e-3, grad=g2)
    assert torch.equal(g2, g) and torch.equal(loss2, loss)
    assert float((prop.params - p0).abs().max()) <= 1.01e-3


@pytest.mark.parametrize("mode", ["rgbsum", "l2"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (8, 8), (16, 8)])
def test_objective_by_regions_and_by_quadrants(mode, tile):
    """The full and fixed objectives of one call by regions (more than 32 768,
    ragged view sizes) and of the same views in calls by quadrants: the same
    bits per ray and per view."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(8000, 24, 1)
    per_view = -(-636 // max(16, tile[0])) * -(-412 // max(16, tile[1])) * max(1, 256 // (tile[0] * tile[1]))
    n_views = 33_000 // per_view + 15
    vw = synth.make_orbit_views(n_views, 25, 636, 412)
    d = gs.DeviceScene.from_scene(sc)
    rng = np.random.default_rng(0)
    wt = torch.as_tensor(rng.exponential(size=8000) * (rng.random(8000) < 0.3)).cuda()
    qm = {"rgbsum": gs.QUERY_RGBSUM, "l2": gs.QUERY_L2}[mode]
    for weights, objective in ((None, gs.OBJ_FULL), (wt, gs.OBJ_FULL), (wt, gs.OBJ_FIXED)):
        kw = dict(query_mode=qm, diag=False, tile=tile)
        every = gs.render_objective(d, vw, weights, objective, **kw)
        each = gs.render_objective(d, vw, weights, objective, max_views_per_chunk=1, **kw)
        assert float(every["per_ray"].max()) > 0
        assert torch.equal(every["per_ray"], each["per_ray"])
        assert torch.equal(every["per_view"], each["per_view"])


@pytest.mark.parametrize("size", [(2048, 40), (2049, 40), (40, 2048), (40, 2049), (1024, 24), (1025, 24)])
def test_ranges_in_half_tiles_and_in_pixels(size):
    """Views of 128 and 129 tiles along an axis (ranges in half tiles, a byte
    each, and in pixels): tiles of 8, 16 and 32 pixels give the same bits, with
    and without a ray mask."""
    import synth
    import paper_2607_02721_amd as gs
    W, H = size
    sc = synth.make_cluster_scene(4000, 26, 1)
    vw = synth.make_orbit_views(2, 27, W, H)
    rng = np.random.default_rng(W + H)
    keep = rng.random((2, H, W)) < 0.002
    mask = torch.as_tensor(synth.pack_bits(keep.reshape(-1)).view(np.int32)).cuda()
    d = gs.DeviceScene.from_scene(sc)
    whole = masked = None
    for tile in ((8, 8), (16, 16), (32, 32)):
        s, _ = gs.sensitivity(d, vw, tile=tile)
        m, _ = gs.sensitivity(d, vw, ray_mask=mask, tile=tile)
        assert float(s.max()) > 0
        assert whole is None or torch.equal(s, whole)
        assert masked is None or torch.equal(m, masked)
        whole, masked = s, m


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8193])
def test_depth_sort_tile_edges(n):
    """Sort tiles of 4096 keys with a last one full, nearly empty and nearly
    full, at the parity bar of 1e-5 against the FP64 oracle."""
    import synth
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    sc = synth.make_cluster_scene(n, 28, 1)
    vw = synth.make_orbit_views(2, 29, 40, 24)
    ref = ora.sensitivity(sc, vw)
    mask_np = synth.pack_bits(~ref["flag"])
    ref = ora.sensitivity(sc, vw, None, mask_np)
    s, _ = gs.sensitivity(gs.DeviceScene.from_scene(sc), vw,
                          ray_mask=torch.as_tensor(mask_np.view(np.int32)).cuda())
    err = np.abs(s.cpu().numpy().astype(np.float64) - ref["s"]) - (1e-5 * ref["s"] + 1e-12)
    assert err.max() <= 0


def test_depth_sort_many_tiles():
    """8200 sort tiles in one call (histograms of four tiles per block) and the
    same views 64 to a chunk (one tile per block)."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(4097, 30, 1)
    vw = synth.make_orbit_views(4100, 31, 8, 8)
    d = gs.DeviceScene.from_scene(sc)
    every, _ = gs.sensitivity(d, vw)
    some, _ = gs.sensitivity(d, vw, max_views_per_chunk=64)
    assert float(every.max()) > 0
    assert torch.equal(every, some)


# blocks of 2048 quanta and their neighbours, a block of zeros in the middle, more
# than 1024 blocks (a thread then takes several of their sums), one Gaussian
@pytest.mark.parametrize("n", [1, 2, 2047, 2048, 2049, 6144, 2_100_000])
@pytest.mark.parametrize("noalloc", [False, True])
def test_sampler_block_edges(n, noalloc):
    """Counts, weights and support equal the oracle's bit for bit; an invalid
    value in any block leaves them all at zero."""
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    rng = np.random.default_rng(n)
    s = rng.uniform(0, 1, n).astype(np.float32)
    s[rng.uniform(size=n) < 0.3] = 0
    s[2048:4096] = 0
    s[-1] = np.float32(0.5)
    ref = ora.sample(s, 5000, 7)
    out = (torch.full((n,), 3, dtype=torch.int32).cuda(), torch.full((n,), 3.0, dtype=torch.float64).cuda(),
           torch.full((1,), 3, dtype=torch.int64).cuda())
    counts, w, sup = gs.sample_coreset(torch.as_tensor(s).cuda(), 5000, 7, out=out, noalloc=noalloc)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), ref["counts"])
    assert np.array_equal(w.cpu().numpy().view(np.uint64), ref["weights"].view(np.uint64))
    assert int(sup.item()) == ref["support"]
    for where in (0, n // 2, n - 1):
        x = s.copy()
        x[where] = -1
        with pytest.raises(gs.GsError):
            gs.sample_coreset(torch.as_tensor(x).cuda(), 5000, 7, out=out, noalloc=noalloc)
        assert not out[0].any() and not out[1].any() and int(out[2]) == 0


@pytest.mark.parametrize("tiles", [(16_384, 1), (16_385, 1), (1, 1)])
def test_list_offsets_of_few_and_many_tiles(tiles):
    """Tile counts at the edge of the one-block scan (as views of one tile):
    a call equals its views 4096 to a chunk, which take that form."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(300, 32, 1)
    vw = synth.make_orbit_views(tiles[0], 33, 16, 16)
    d = gs.DeviceScene.from_scene(sc)
    every, _ = gs.sensitivity(d, vw)
    some, _ = gs.sensitivity(d, vw, max_views_per_chunk=4096)
    assert float(every.max()) > 0
    assert torch.equal(every, some)


@pytest.mark.parametrize("n", [1, 64, 1023, 1024, 1025, 3000, 4096])
@pytest.mark.parametrize("far", [False, True])
def test_one_block_sort(n, far):
    """Segments of up to 4096 keys, over three passes and (depths over more than
    two octaves) four, of all Gaussians and of the kept ones of a ray mask, at the
    parity bar of 1e-5 against the FP64 oracle."""
    import synth
    import paper_2607_02721_amd as gs
    from oracle import oracle as ora
    ora.build(force=False)
    sc = synth.make_cluster_scene(n, 34, 1)
    if far:
        sc.mean *= np.float32(1) + np.float32(40) * (np.arange(n) % 3 == 0).astype(np.float32)
    vw = synth.make_orbit_views(3, 35, 96, 40)
    ref = ora.sensitivity(sc, vw)
    keep = ~ref["flag"]
    few = keep.reshape(3, 40, 96).copy()
    few[:, :, 24:] = False
    for sel in (keep, few.reshape(-1)):
        bits = synth.pack_bits(sel)
        want = ora.sensitivity(sc, vw, None, bits)["s"]
        s, _ = gs.sensitivity(gs.DeviceScene.from_scene(sc), vw,
                              ray_mask=torch.as_tensor(bits.view(np.int32)).cuda())
        err = np.abs(s.cpu().numpy().astype(np.float64) - want) - (1e-5 * want + 1e-12)
        assert err.max() <= 0


@pytest.mark.parametrize("n", [1500, 2100, 9000])
@pytest.mark.parametrize("masked", [False, True])
def test_emission_carries_positions_between_batches(n, masked):
    """Chunks of several batches (200 views in one call take chunks of up to
    2^14 positions, queued 1024 or, with a ray mask, 2048 at a time) whose rows
    meet few positions each, so that batches leave positions over: one call of
    all views is the maximum of calls of one view, whose chunks are one batch."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(n, 36, 0)
    sc.log_scale[:] -= np.float32(1.5)
    vw = synth.make_orbit_views(400, 37, 48, 1600)
    d = gs.DeviceScene.from_scene(sc)
    keep = np.ones((400, 1600, 48), bool)
    if masked:
        keep[:, ::2, :] = False
    mask = lambda k: torch.as_tensor(synth.pack_bits(k.reshape(-1)).view(np.int32)).cuda() if masked else None
    every, _ = gs.sensitivity(d, vw, ray_mask=mask(keep))
    each = torch.zeros_like(every)
    for v in range(400):
        each = torch.maximum(each, gs.sensitivity(d, vw.subset([v]), ray_mask=mask(keep[v]))[0])
    assert float(every.max()) > 0
    assert torch.equal(every, each)


@pytest.mark.parametrize("aggregate", ["ray", "image"])
def test_many_regions_in_tile_order(aggregate):
    """132 600 regions of one scene composite in tile order, 52 000 at a time by
    descending list length (or by quadrants): the same sensitivities."""
    import synth
    import paper_2607_02721_amd as gs
    sc = synth.make_cluster_scene(3000, 38, 1)
    vw = synth.make_orbit_views(510, 39, 320, 208)
    d = gs.DeviceScene.from_scene(sc)
    agg = {"ray": gs.AGG_RAY, "image": gs.AGG_IMAGE}[aggregate]
    every, _ = gs.sensitivity(d, vw, aggregate=agg)
    some, _ = gs.sensitivity(d, vw, aggregate=agg, max_views_per_chunk=200)
    assert float(every.max()) > 0
    assert torch.equal(every, some)
