"""Loop-closure grid search (Section III-C): candidate transforms scored by
the number of Omega inliers at a coarse pyramid level, the best one promoted
to the full-resolution batched registration.

Scores are compared with the FP64 oracle's inlier counts at the same
candidate poses on identical inputs (the oracle's surfel images, rounded to
FP32, on both sides): each integer score within the number of pixels whose
FP64 projection or gate value lies at a boundary, the winner the oracle's
wherever its margin exceeds that; the promoted registrations are compared
with identity-started ones on pairs with relative yaw up to 90 deg."""
import math

import numpy as np
import pytest

import oracle as O
import synth
from parity_checks import association_ambiguous, assert_scores_match
from synth import workloads as W

pytestmark = pytest.mark.gpu

BATCH_PARAMS = dict(levels=3, iters=(10, 10, 10), stop_update_norm=1e-6)


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _candidate(c, n_yaw, n_xy, step):
    """G_c written out from its definition (FP64, 4x4)."""
    a, u, v = c // (n_xy * n_xy), (c // n_xy) % n_xy, c % n_xy
    h = (n_xy - 1) / 2
    return synth.se3(synth.rot_z(2 * math.pi * a / n_yaw), [(u - h) * step, (v - h) * step, 0.0])


def _oracle_items(pairs):
    """Items carrying the oracle's level-0 surfel images (FP32) of each pair;
    returns the items and, per pair, the level-2 images of both (FP64 copies
    of the same FP32 values)."""
    items, lvl2 = [], []
    for p in pairs:
        g = p["geom"]
        s32 = O.panorama_normals(g, p["scan"]).astype(np.float32)
        k32 = O.panorama_normals(g, p["kf"]).astype(np.float32)
        items.append(dict(scan_geom=g, kf_geom=g, scan_surfel=_t(s32), kf_surfel=_t(k32)))
        lvl2.append((O.pyramid_level(g, s32.astype(np.float64), 2), O.pyramid_level(g, k32.astype(np.float64), 2)))
    return items, lvl2


def _check_scores(g, sl, kl, scores_k, poses, d_max):
    gl = g.level(2)
    cos_t = math.cos(math.radians(30.0))
    ref = np.array([int(O.correspondences(gl, sl, gl, kl, T, d_max, cos_t)[1].sum()) for T in poses])
    amb = np.array([int(association_ambiguous(gl, sl, gl, kl, T, d_max, cos_t).sum()) for T in poses])
    return assert_scores_match(scores_k, ref, amb)


def _items(pairs):
    import torch
    items = []
    for p in pairs:
        g = p["geom"]
        items.append(dict(scan_geom=g, kf_geom=g, scan_depth=_t(p["scan"]), kf_depth=_t(p["kf"]),
                          scan_surfel=torch.empty((g.rows, g.cols, 4), dtype=torch.float32, device="cuda"),
                          kf_surfel=torch.empty((g.rows, g.cols, 4), dtype=torch.float32, device="cuda")))
    return items


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context(0, max_pixels=128 * 2048, max_batch=64, max_batch_pixels=64 * 128 * 2048)
    yield c
    c.close()


# (n_yaw, n_xy): the per-yaw kernels (1 to 5 grid cells per axis, yaw chunks
# that do not divide n_yaw included) and the general kernel (6 cells per axis)
@pytest.mark.parametrize("n_yaw,n_xy", [(12, 3), (7, 1), (5, 2), (3, 4), (2, 5), (2, 6)])
def test_scores_match_oracle_counts(gpu_lib, ctx, n_yaw, n_xy):
    pairs = [W.batch_pair(k, base_seed=5_000_000, max_angle=math.radians(90.0), size=(64, 512)) for k in range(2)]
    gp = gpu_lib.GridParams(level=2, n_yaw=n_yaw, n_xy=n_xy, xy_step=0.7, d_max=2.0)
    items, lvl2 = _oracle_items(pairs)
    b = gpu_lib.Batch(ctx, items, gpu_lib.IcpParams(**BATCH_PARAMS))
    best, best_score, scores = b.grid_search(gp)
    scores = scores.cpu().numpy()
    best = best.cpu().numpy()
    best_score = best_score.cpu().numpy()
    C = n_yaw * n_xy * n_xy
    assert scores.shape == (len(pairs), C)
    for k, p in enumerate(pairs):
        sl, kl = lvl2[k]
        dev, amb = _check_scores(p["geom"], sl, kl, scores[k], [_candidate(c, n_yaw, n_xy, 0.7) for c in range(C)],
                                 2.0)
        print(f"pair {k}: {C} candidates, total |score - oracle| {dev}, ambiguous pixels {amb}")
        c_best = int(np.argmax(scores[k]))
        assert best_score[k] == scores[k].max() and np.argmax(scores[k] == scores[k].max()) == c_best
        T = np.eye(4)
        T[:3, :3] = best[k, :9].reshape(3, 3)
        T[:3, 3] = best[k, 9:]
        np.testing.assert_allclose(T, _candidate(c_best, n_yaw, n_xy, 0.7), atol=1e-12)
    b.close()


def test_grid_start_beats_identity_at_large_yaw(gpu_lib, ctx):
    import torch
    n = 32
    pairs = [W.batch_pair(k, base_seed=5_100_000, max_angle=math.radians(90.0), max_trans=2.0) for k in range(n)]
    items = _items(pairs)
    b = gpu_lib.Batch(ctx, items, gpu_lib.IcpParams(**BATCH_PARAMS))
    b.normals()
    plain = gpu_lib.read_results(b.register([np.eye(4)] * n))
    best, _, _ = b.grid_search(gpu_lib.GridParams())
    grid = gpu_lib.read_results(b.register(best))
    torch.cuda.synchronize()

    def ok(res):
        return np.array([synth.pose_error(r["T"], p["T_gt"])[0] < math.radians(1.0)
                         and synth.pose_error(r["T"], p["T_gt"])[1] < 0.05 for r, p in zip(res, pairs)])

    s_plain, s_grid = ok(plain), ok(grid)
    print(f"\ngrid search: success identity start {s_plain.sum()}/{n}, grid start {s_grid.sum()}/{n}")
    assert s_grid.sum() >= s_plain.sum() + 0.1 * n
    assert s_grid.mean() >= 0.8
    b.close()


def test_grid_search_replays_from_a_graph(gpu_lib, ctx):
    import torch
    pairs = [W.batch_pair(k, base_seed=5_200_000, max_angle=math.radians(60.0), size=(64, 512)) for k in range(4)]
    items = _items(pairs)
    b = gpu_lib.Batch(ctx, items, gpu_lib.IcpParams(**BATCH_PARAMS))
    gp = gpu_lib.GridParams(n_yaw=18)
    base = torch.stack([gpu_lib.pose_tensor(np.eye(4)) for _ in items])
    scores = torch.empty((4, 18 * 9), dtype=torch.int32, device="cuda")
    best = torch.empty((4, 12), dtype=torch.float64, device="cuda")
    bsc = torch.empty(4, dtype=torch.int32, device="cuda")
    b.normals()
    b.grid_search(gp, base, scores, best, bsc)
    torch.cuda.synchronize()
    eager = (scores.cpu().numpy().copy(), best.cpu().numpy().copy())
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        b.grid_search(gp, base, scores, best, bsc)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            b.grid_search(gp, base, scores, best, bsc)
    for _ in range(2):
        scores.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(scores.cpu().numpy(), eager[0]) and np.array_equal(best.cpu().numpy(), eager[1])
    b.close()


def test_scores_around_a_base_pose(gpu_lib, ctx):
    """The candidates are base * G_c: scores against the oracle's counts at
    base * G_c for a base pose per registration."""
    import torch
    pairs = [W.batch_pair(k, base_seed=5_100_000, max_angle=math.radians(40.0), size=(64, 512)) for k in range(2)]
    bases = [synth.se3(synth.rot_z(0.3 + k), [0.5, -0.2 * k, 0.05]) for k in range(2)]
    gp = gpu_lib.GridParams(level=2, n_yaw=4, n_xy=3, xy_step=0.5, d_max=2.0)
    items, lvl2 = _oracle_items(pairs)
    b = gpu_lib.Batch(ctx, items, gpu_lib.IcpParams(**BATCH_PARAMS))
    base_t = torch.stack([gpu_lib.pose_tensor(T) for T in bases])
    best, _, scores = b.grid_search(gp, base_t)
    scores = scores.cpu().numpy()
    for k, p in enumerate(pairs):
        sl, kl = lvl2[k]
        _check_scores(p["geom"], sl, kl, scores[k], [bases[k] @ _candidate(c, 4, 3, 0.5) for c in range(36)], 2.0)
        c_best = int(np.argmax(scores[k]))
        T = np.eye(4)
        T[:3, :3] = best.cpu().numpy()[k, :9].reshape(3, 3)
        T[:3, 3] = best.cpu().numpy()[k, 9:]
        np.testing.assert_allclose(T, bases[k] @ _candidate(c_best, 4, 3, 0.5), atol=1e-12)
    b.close()


@pytest.mark.parametrize("half", [22.5, 44.5, 70.0])
def test_keyframe_tables_give_the_general_kernels_scores(gpu_lib, half):
    """The per-yaw kernels read the keyframe from a table of points at levels 1
    and up, with a projection of their own; the kernel for more than 5 grid cells
    per axis reads the images and projects as everywhere else.  A 7 x 7 grid
    holds the candidates of the 3 x 3 and 1 x 1 grids of the same step: equal
    scores, for a panorama within +-45 deg and ones that reach past it, with
    holes, bases of any heading (azimuths on both sides of the seam) and points
    next to the axes."""
    import torch
    rng = np.random.Generator(np.random.PCG64(int(half)))
    rows, cols = 24, 512
    g = synth.Geom(rows, cols, math.radians(half), math.radians(2 * half) / (rows - 1))
    ctx = gpu_lib.Context(0, max_pixels=rows * cols, max_batch=4, max_batch_pixels=4 * rows * cols)
    items, base = [], []
    for k in range(4):
        el = g.el_top - g.d_el * np.arange(rows)[:, None]
        az = 2 * np.pi * np.arange(cols)[None, :] / cols
        # a 12 x 8 x 5 m box around the sensor, 2 cm noise, a tenth of the returns missing
        u = np.stack([np.cos(el) * np.cos(az), np.cos(el) * np.sin(az), np.sin(el) + 0 * az], -1)
        t = np.min(np.where(u > 0, np.array([6, 4, 3.0]), np.array([-6, -4, -2.0])) / np.where(u == 0, 1e-9, u), -1)
        images = []
        for _ in range(2):
            d = t + 0.02 * rng.normal(size=t.shape)
            d[rng.uniform(size=t.shape) < 0.1] = 0.0
            images.append(gpu_lib.panorama_normals(ctx, g, torch.from_numpy(d.astype(np.float32)).cuda()))
        items.append(dict(scan_geom=g, kf_geom=g, scan_surfel=images[0], kf_surfel=images[1]))
        base.append(gpu_lib.pose_tensor(synth.se3(synth.rot_z(k * np.pi / 2 + (k > 1) * 0.3), [0.1 * k, 0, 0])))
    b = gpu_lib.Batch(ctx, items, gpu_lib.IcpParams(levels=3, iters=(1, 1, 1, 0)))
    base = torch.stack(base)
    for level in (0, 1, 2):
        def score(n_xy):
            gp = gpu_lib.GridParams(level=level, n_yaw=12, n_xy=n_xy, xy_step=0.5, d_max=1.0)
            return b.grid_search(gp, base)[2].cpu().numpy().reshape(4, 12, n_xy, n_xy)
        full = score(7)
        assert full.max() > 0.2 * (rows >> level) * (cols >> level)
        assert np.array_equal(score(3), full[:, :, 2:5, 2:5])
        assert np.array_equal(score(5), full[:, :, 1:6, 1:6])
        assert np.array_equal(score(1), full[:, :, 3:4, 3:4])
    b.close()
    ctx.close()


def test_points_of_denormal_range_project_nowhere(gpu_lib):
    """Surfels whose ranges are denormal are valid where the sensor has no
    minimum range, and the azimuth and elevation of such a point are no numbers:
    outside +-45 deg they count for no candidate, with the table as with the
    images (7 x 7), although a keyframe 0.5 m away lies within reach."""
    import torch
    rows, cols = 24, 512
    g = synth.Geom(rows, cols, math.radians(70.0), math.radians(140.0) / (rows - 1))
    assert g.r_min == 0.0
    el = g.el_top - g.d_el * np.arange(rows)[:, None]
    az = 2 * np.pi * np.arange(cols)[None, :] / cols
    u = np.stack([np.cos(el) * np.cos(az), np.cos(el) * np.sin(az), np.sin(el) + 0 * az], -1)
    kf = np.concatenate([-u, np.full(u.shape[:2] + (1,), 0.5)], -1).astype(np.float32)
    scan = kf.copy()
    scan[:, ::8, 3] = np.float32(1e-39)  # every second pixel of level 2, the columns of the axes among them
    assert scan[0, 0, 3] > 0
    ctx = gpu_lib.Context(0, max_pixels=rows * cols, max_batch=1, max_batch_pixels=rows * cols)
    b = gpu_lib.Batch(ctx, [dict(scan_geom=g, kf_geom=g, scan_surfel=_t(scan), kf_surfel=_t(kf))],
                      gpu_lib.IcpParams(levels=3, iters=(1, 1, 1, 0)))
    base = torch.stack([gpu_lib.pose_tensor(np.eye(4))])
    for level in (1, 2):
        def score(n_xy):
            gp = gpu_lib.GridParams(level=level, n_yaw=12, n_xy=n_xy, xy_step=0.0, d_max=1.0)
            return b.grid_search(gp, base)[2].cpu().numpy().reshape(12, n_xy, n_xy)
        full = score(7)
        usable = np.count_nonzero(scan[::1 << level, ::1 << level, 3] == 0.5)
        assert (full[0] == usable).all()
        assert np.array_equal(score(3), full[:, 2:5, 2:5])
        assert np.array_equal(score(1), full[:, 3:4, 3:4])
    b.close()
    ctx.close()


def test_keyframe_tables_take_the_normals_scratch(gpu_lib):
    """A batch whose items have depth images lays the grid search's tables out
    in its scratch for normals: it takes the memory of the normals (16 bytes a
    pixel) less the tables (24 bytes an entry) more than a batch of the same
    surfel images alone, and a search between normals and registrations
    changes neither."""
    import torch
    n, rows, cols, levels = 48, 128, 2048, 3
    pair = W.batch_pair(0, base_seed=5_500_000, max_angle=math.radians(20.0), size=(rows, cols))
    g = pair["geom"]
    ctx = gpu_lib.Context(0, max_pixels=rows * cols, max_batch=n, max_batch_pixels=n * rows * cols)
    full = _items([pair] * n)
    bare = [{k: v for k, v in it.items() if "depth" not in k} for it in full]
    params = gpu_lib.IcpParams(levels=levels, iters=(4, 4, 4))
    taken = {}
    gp = gpu_lib.GridParams(level=1, n_yaw=12, n_xy=2, xy_step=0.5, d_max=1.0)
    found = {}
    for name, items in (("warm", full), ("depth", full), ("bare", bare)):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        b = gpu_lib.Batch(ctx, items, params)
        torch.cuda.synchronize()
        taken[name] = before - torch.cuda.mem_get_info()[0]
        if name == "depth":
            b.normals()
            plain = b.register([np.eye(4)] * n).cpu().numpy()
            b.grid_search(gp)
            b.normals()
            again = b.register([np.eye(4)] * n).cpu().numpy()
            assert np.array_equal(plain, again)
        found[name] = b.grid_search(gp)[2].cpu().numpy()
        b.close()
    ctx.close()
    assert found["depth"].max() > 0 and np.array_equal(found["depth"], found["bare"])
    normals = 2 * n * rows * cols * 16
    tables = sum(n * ((rows >> l) * ((cols >> l) + 1) + 1) * 24 for l in range(1, levels))
    print(f"[grid] {taken['depth'] / 2**20:.1f} MiB with depth images, {taken['bare'] / 2**20:.1f} without, "
          f"normals {normals / 2**20:.1f}, tables {tables / 2**20:.1f}")
    # the normals' lists of tiles, and the allocator's granularity of 2 MiB in a few allocations
    assert taken["depth"] - taken["bare"] <= normals - tables + (16 << 20)


def test_searches_with_and_without_tables(gpu_lib):
    """Whether a search takes the keyframes' tables depends on its candidates
    and on the batch's sizes; its scores do not: 12 yaws (images) and the same
    with four equal translations (tables); scans of half the keyframe's columns
    in a batch of two (tables of 3.2 MB) and of three (images)."""
    pairs = [W.batch_pair(k, base_seed=5_600_000, max_angle=math.radians(40.0), size=(128, 2048)) for k in range(3)]
    ctx = gpu_lib.Context(0, max_pixels=128 * 2048, max_batch=3, max_batch_pixels=3 * 128 * 2048)
    items = _items(pairs)
    for it in items:
        gpu_lib.panorama_normals(ctx, it["scan_geom"], it["scan_depth"], it["scan_surfel"])
        gpu_lib.panorama_normals(ctx, it["kf_geom"], it["kf_depth"], it["kf_surfel"])
    half = []
    for it in items:
        g = it["scan_geom"]
        h = synth.Geom(g.rows, g.cols // 2, g.el_top, g.d_el, g.r_min, g.r_max)
        half.append(dict(it, scan_geom=h, scan_surfel=it["scan_surfel"][:, ::2].contiguous(), scan_depth=None))
    params = gpu_lib.IcpParams(levels=3, iters=(1, 1, 1))
    for group in (items, half):
        b = gpu_lib.Batch(ctx, group, params)
        for level in (1, 2):
            one, four = (b.grid_search(gpu_lib.GridParams(level=level, n_yaw=12, n_xy=k, xy_step=0.0, d_max=1.0))[2]
                         .cpu().numpy().reshape(3, 12, k * k) for k in (1, 2))
            assert one.max() > 100 and np.array_equal(np.repeat(one, 4, axis=2), four)
        b.close()
    scores = []
    for group in (half[:2], half):
        b = gpu_lib.Batch(ctx, group, params)
        gp = gpu_lib.GridParams(level=1, n_yaw=36, n_xy=2, xy_step=0.5, d_max=1.0)
        scores.append(b.grid_search(gp)[2].cpu().numpy()[:2])
        b.close()
    assert scores[0].max() > 100 and np.array_equal(*scores)
    ctx.close()
