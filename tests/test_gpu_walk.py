"""The backward's walk over a block's records: list lengths around its steps of
four and its chunks of 64, both widths of the gradient sums, and what a
non-finite upstream gradient reaches. Bars as in test_gpu_parity."""
import numpy as np
import pytest

import oracle
from paper_2312_10070_amd import gsr
from tests import gpu_cases as G
from tests import helpers as H

pytestmark = pytest.mark.gpu

CAM = oracle.Camera(19, 11, 20.0, 20.0, 9.0, 5.0, 0.2, (0.1, 0.2, 0.3))  # ragged: two tiles, cut blocks
POSE = np.array([1, 0, 0, 0, 0, 0, 0], np.float64)


def stack(m, n, seed):
    """m Gaussians over the image at well separated depths (opacities low enough that no pixel stops early),
    the other n - m behind the camera."""
    rng = np.random.default_rng(seed)
    z = 1.0 + 0.03 * np.arange(n)
    g = dict(means=np.stack([rng.uniform(-0.3, 0.3, n) * z, rng.uniform(-0.2, 0.2, n) * z, z], 1),
             scales=rng.uniform(0.05, 0.2, (n, 3)) * z[:, None], quats=rng.normal(size=(n, 4)),
             opacities=rng.uniform(0.02, 0.05, n), colors=rng.uniform(0, 1, (n, 3)))
    g["means"][m:, 2] = -1.0
    return G.certify(g, POSE, CAM, 1e-4) if n <= 1000 else G.f32(g)


def backward(g, gC, gD, **kw):
    import torch
    d = G.to_dev(g)
    camera = gsr.make_camera(CAM.width, CAM.height, CAM.fx, CAM.fy, CAM.cx, CAM.cy, CAM.near_z, CAM.bg)
    pose = torch.tensor(POSE.astype(np.float32), device="cuda")
    _, _, _, st = gsr.render_fwd(d["means"], d["scales"], d["quats"], d["opacities"], d["colors"], pose, camera)
    out = gsr.render_bwd(st, torch.from_numpy(gC).cuda(), torch.from_numpy(gD).cuda(), None, **kw)
    torch.cuda.synchronize()
    st.release()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("m", [1, 3, 4, 5, 63, 64, 65, 67, 68, 129])
@pytest.mark.parametrize("n", [None, 40000])  # n <= 32768: sums in double, above: in float
def test_walk_lengths(m, n):
    g = stack(m, m if n is None else n, m)
    rng = np.random.default_rng(m + 1)
    gC = rng.normal(size=(3, CAM.height, CAM.width)).astype(np.float32)
    gD = rng.normal(size=(CAM.height, CAM.width)).astype(np.float32)
    vis = {k: v[:m] for k, v in g.items()}
    ref = oracle.backward(vis, POSE, CAM, oracle.Opts(amb_z=0.0), gC, gD)
    full = backward(g, gC, gD)
    if n is not None:
        assert all(not np.any(full[k][m:]) for k in gsr.PARAM_GROUPS)
    G.grads_check({k: full[k][:m] for k in gsr.PARAM_GROUPS}, ref, case=f"walk {m}")
    pose_only = backward(g, gC, gD, want_params=False)
    for out in (full, pose_only):
        for k in ("pose7", "twist6"):
            H.check_grad_ref(k, out[k], ref, case=f"walk {m}")


def test_non_finite_upstream_stays_in_its_pixel():
    """A NaN upstream gradient at one pixel: the geometry of records of the same step of the walk that do not
    cover the pixel is not touched by it, and blocks without the pixel not at all."""
    n = 8
    g = dict(means=np.zeros((n, 3)), scales=np.full((n, 3), 0.02), quats=np.tile([1.0, 0, 0, 0], (n, 1)),
             opacities=np.full(n, 0.3), colors=np.full((n, 3), 0.5))
    z = 1.0 + 0.05 * np.arange(n)
    # alternately around pixel (2, 2), around pixel (6, 6) of the same block, and in another block
    px = np.array([2, 6, 2, 6, 13, 6, 2, 13], np.float64)
    py = np.array([2, 6, 2, 6, 3, 6, 2, 3], np.float64)
    g["means"] = np.stack([(px - CAM.cx) / CAM.fx * z, (py - CAM.cy) / CAM.fy * z, z], 1)
    g["scales"] = np.full((n, 3), 0.02)
    gC = np.full((3, CAM.height, CAM.width), 0.5, np.float32)
    gD = np.full((CAM.height, CAM.width), 0.25, np.float32)
    want = backward(G.f32(g), gC, gD, want_pose=False)
    gC[1, 2, 2] = np.nan
    got = backward(G.f32(g), gC, gD, want_pose=False)
    clean = px != 2
    assert np.isnan(got["means"][~clean]).all()
    for k in ("means", "scales", "quats", "opacities"):
        np.testing.assert_array_equal(got[k][clean], want[k][clean], err_msg=k)
    np.testing.assert_array_equal(got["colors"][px == 13], want["colors"][px == 13])


@pytest.mark.parametrize("ntx,nty", [(16, 16), (257, 1), (64, 128), (211, 39)])
def test_every_tile_is_rendered_in_any_order(ntx, nty):
    """Tile counts around the 256 up to which the tiles keep their order and the
    8,192 the ordering takes at a time, lists of 0 to a few hundred: one pixel
    of every tile against the oracle (the bar of test_gpu_fullsize)."""
    import torch
    W, Hh, n_tiles = 16 * ntx, 16 * nty, ntx * nty
    cam = oracle.Camera(W, Hh, 400.0, 400.0, W / 2, Hh / 2, 0.2, (0.0, 0.0, 0.0))
    rng = np.random.default_rng(n_tiles)
    tile = np.concatenate([np.flatnonzero(rng.uniform(size=n_tiles) < 0.9), np.full(300, n_tiles // 3),
                           rng.integers(0, n_tiles, 2000)])
    n = len(tile)
    u, v = 16 * (tile % ntx) + 8, 16 * (tile // ntx) + 8
    z = 2.0 + 1e-3 * rng.permutation(n)
    g = G.f32(dict(means=np.stack([(u - W / 2) / 400 * z, (v - Hh / 2) / 400 * z, z], 1),
                   scales=np.repeat((rng.uniform(0.5, 1.5, n) * z / 400)[:, None], 3, 1),
                   quats=np.tile([1.0, 0, 0, 0], (n, 1)), opacities=rng.uniform(0.02, 0.4, n),
                   colors=rng.uniform(0, 1, (n, 3))))
    d = G.to_dev(g)
    color, depth, alpha, st = gsr.render_fwd(d["means"], d["scales"], d["quats"], d["opacities"], d["colors"],
                                             torch.tensor(POSE.astype(np.float32), device="cuda"),
                                             gsr.make_camera(W, Hh, 400.0, 400.0, W / 2, Hh / 2, 0.2))
    torch.cuda.synchronize()
    st.release()
    t = np.arange(n_tiles)
    yy, xx = 16 * (t // ntx) + 8, 16 * (t % ntx) + 8
    orc = oracle.render(g, POSE, cam, oracle.Opts(amb_rel=2e-4, amb_z=5e-7), pixels=yy * W + xx, nthreads=8)
    pick = lambda a: a[..., yy, xx]
    G.compare_images({k: pick(a.cpu().numpy()) for k, a in (("color", color), ("depth", depth), ("alpha", alpha))},
                     {k: pick(a) for k, a in orc.items() if k != "hash"}, dict(color=1e-4, depth=1e-4, alpha=1e-4),
                     max_unverifiable=0.02)


@pytest.mark.parametrize("V", [3, 6, 33])
def test_lists_by_length_give_what_lists_in_place_give(V):
    """Views of 256 tiles: one by one their lists are taken as they lie; as one
    batch (768 items: rounds reversed; 1,536; 8,448: ordered in two stretches)
    by length. A tile's pixels do not depend on the order, so the images are
    equal to the bit."""
    import torch
    rng = np.random.default_rng(V)
    n = 20000
    z = rng.uniform(2.0, 4.0, n)
    g = G.to_dev(dict(means=np.stack([rng.uniform(-0.35, 0.35, n) * z, rng.uniform(-0.35, 0.35, n) * z, z], 1),
                      scales=np.repeat((rng.uniform(2.0, 12.0, n) * z / 400)[:, None], 3, 1),
                      quats=np.tile([1.0, 0, 0, 0], (n, 1)), opacities=rng.uniform(0.02, 0.9, n),
                      colors=rng.uniform(0, 1, (n, 3))))
    args = [g[k] for k in ("means", "scales", "quats", "opacities", "colors")]
    camera = gsr.make_camera(256, 256, 400.0, 400.0, 128.0, 128.0, 0.2)
    poses = np.tile(POSE, (V, 1))
    poses[:, 4] = np.linspace(-0.2, 0.2, V)
    poses = torch.from_numpy(poses.astype(np.float32)).cuda()
    cb, db, ab, st = gsr.render_fwd_batch(*args, poses, camera, gsr.RasterOpts())
    K = gsr.tile_lists(st, 256 * V)[0]
    st.release()
    assert 1 << 18 <= K < V << 18  # by length as one batch, as they lie one by one
    for v in range(V):
        c, d, a, st = gsr.render_fwd(*args, poses[v].contiguous(), camera)
        assert gsr.tile_lists(st, 256)[0] < 1 << 18
        st.release()
        assert torch.equal(cb[v], c) and torch.equal(db[v], d) and torch.equal(ab[v], a)


@pytest.mark.parametrize("lengths", [[255, 256, 257, 511, 512, 1536, 1537, 1025, 2],
                                     [2048, 2049, 3073, 1024, 1025, 256, 257, 4097, 3]])
def test_sort_networks_and_runs(lengths):
    """Lists around the 256-key network and the runs of 512 (mean length below
    1,024), and around the 2048-key network and the runs of 1,024 (above):
    bit-exact against the oracle, with depth ties."""
    from tests.test_gpu_parity import run_fwd, tile_stacks
    g, cam = tile_stacks(lengths, seed=3)
    g = G.certify(g, POSE, cam, 1e-4)
    tl = oracle.tile_lists(g, POSE, cam, oracle.Opts())
    assert (tl["ranges"][:, 1] - tl["ranges"][:, 0]).tolist() == lengths
    _, st, _, _ = run_fwd(g, POSE, cam)
    K, ranges, ids = gsr.tile_lists(st, 9)
    assert K == sum(lengths)
    G.compare_tile_lists(ranges.cpu().numpy(), ids.cpu().numpy(), tl, None)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("which", ["color", "depth"])
@pytest.mark.parametrize("n", [8, 40000])
def test_non_finite_upstream_reaches_what_its_pixel_composited(bad, which, n):
    """A non-finite upstream gradient at pixel (2, 2), of colour or of depth. The
    gradients of records that pixel (2, 2) did not composite are what they are
    without it, all of them: of records in the same steps of the walk around
    another pixel of the block, of one (the seventh) that passes the block's test
    between two pixels and meets none, and of records of another block; in double
    and in float sums (every record lies in one block, so that those have no order)."""
    px = np.array([2, 5, 2, 5, 13, 5, 8.8, 13], np.float64)
    py = np.array([2, 5, 2, 5, 3, 5, 3.5, 3], np.float64)
    z = np.concatenate([1.0 + 0.05 * np.arange(8), np.full(n - 8, -1.0)])
    m = np.zeros((n, 3))
    m[:8, 0], m[:8, 1] = (px - CAM.cx) / CAM.fx * z[:8], (py - CAM.cy) / CAM.fy * z[:8]
    m[:, 2] = z
    g = G.f32(dict(means=m, scales=np.full((n, 3), 0.02), quats=np.tile([1.0, 0, 0, 0], (n, 1)),
                   opacities=np.full(n, 0.3), colors=np.full((n, 3), 0.5)))
    bare = {k: np.delete(v, [0, 2], 0) for k, v in g.items()}  # without the records of the pixel
    gC = np.full((3, CAM.height, CAM.width), 0.5, np.float32)
    gD = np.full((CAM.height, CAM.width), 0.25, np.float32)
    want, pose = backward(g, gC, gD, want_pose=False), backward(bare, gC, gD)
    (gC[1] if which == "color" else gD)[2, 2] = bad
    got = backward(g, gC, gD, want_pose=False)
    reached = np.zeros(n, bool)
    reached[[0, 2]] = True
    for k in gsr.PARAM_GROUPS:
        np.testing.assert_array_equal(got[k][~reached], want[k][~reached], err_msg=k)
    for k in ("means", "opacities"):
        assert not np.isfinite(got[k][reached]).any(), k
    # ten sums and the pose's six, where the pixel composited nothing
    for kw in (dict(), dict(want_params=False)):
        out = backward(bare, gC, gD, **kw)
        for k in ("pose7", "twist6"):
            np.testing.assert_allclose(out[k], pose[k], rtol=1e-5, atol=1e-6 * np.abs(pose[k]).max())


@pytest.mark.parametrize("ntx,nty", [(27, 19), (40, 30), (40, 32), (61, 21), (128, 64), (211, 39)])
def test_tiles_by_length_equal_tiles_in_place(ntx, nty):
    """513, 1,200, 1,280, 1,281, 8,192 and 8,229 tiles with K >= 2^18, which are
    taken by length: two rounds of 256 reversed and one tile more, a partial last
    round, five full rounds, one tile more than rounds are reversed for, one
    stretch of the ordering, and a ragged second. Images and gradients (the
    deterministic option) against those of windows of at most 512 tiles, which
    are taken as they lie, equal to the bit: every Gaussian lies in one tile, all
    coordinates are exact in both frames. (The scenes above have fewer entries,
    and their tiles are taken as they lie.)"""
    import torch
    f, n_tiles = 4096.0, ntx * nty
    rng = np.random.default_rng(n_tiles)
    lengths = rng.integers(0, 2 * (1 << 18) // n_tiles + 40, n_tiles)
    lengths[rng.integers(0, n_tiles, 20)] += 700
    t = rng.permutation(np.repeat(np.arange(n_tiles), lengths))
    n = len(t)
    u = 16 * (t % ntx) + 7.5 + rng.integers(-128, 129, n) / 64
    v = 16 * (t // ntx) + 7.5 + rng.integers(-128, 129, n) / 64
    cx, cy = 8.0 * ntx, 8.0 * nty
    d = G.to_dev(dict(means=np.stack([(u - cx) / f, (v - cy) / f, np.ones(n)], 1),
                      scales=rng.uniform(0.2, 0.8, (n, 3)) / f, quats=rng.normal(size=(n, 4)),
                      opacities=rng.uniform(0.02, 0.4, n), colors=rng.uniform(0, 1, (n, 3))))
    pose = torch.tensor(POSE.astype(np.float32), device="cuda")
    gC = torch.from_numpy(rng.normal(size=(3, 16 * nty, 16 * ntx)).astype(np.float32)).cuda()
    gD = torch.from_numpy(rng.normal(size=(16 * nty, 16 * ntx)).astype(np.float32)).cuda()

    def run(x0, x1, y0, y1):
        camera = gsr.make_camera(16 * (x1 - x0), 16 * (y1 - y0), f, f, cx - 16 * x0, cy - 16 * y0, 0.2)
        sl = (slice(16 * y0, 16 * y1), slice(16 * x0, 16 * x1))
        *img, st = gsr.render_fwd(d["means"], d["scales"], d["quats"], d["opacities"], d["colors"], pose, camera,
                                  gsr.RasterOpts(deterministic=1))
        K = gsr.tile_lists(st, (x1 - x0) * (y1 - y0))[0]
        out = gsr.render_bwd(st, gC[(slice(None), *sl)].contiguous(), gD[sl].contiguous(), want_pose=False)
        st.release()
        return img, out, K, sl

    (color, depth, alpha), grads, K, _ = run(0, ntx, 0, nty)
    assert K == n >= 1 << 18 and n_tiles > 512
    parts = {k: torch.zeros_like(x) for k, x in grads.items()}
    for y0 in range(0, nty, 16):
        for x0 in range(0, ntx, 32):
            img, out, _, sl = run(x0, min(x0 + 32, ntx), y0, min(y0 + 16, nty))
            assert torch.equal(color[(slice(None), *sl)], img[0])
            assert torch.equal(depth[sl], img[1]) and torch.equal(alpha[sl], img[2])
            for k in gsr.PARAM_GROUPS:
                parts[k] += out[k]
    for k in gsr.PARAM_GROUPS:
        assert torch.equal(grads[k], parts[k]) and bool((grads[k] != 0).any()), k
