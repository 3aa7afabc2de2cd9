"""The per-tile depth sort over lengths and launch shapes, and that a call does
not depend on what its context served before."""
import ctypes

import numpy as np
import pytest

from paper_2312_10070_amd import gsr

pytestmark = pytest.mark.gpu

EDGES = [1023, 1024, 1025, 1535, 1536, 1537, 2047, 2048, 2049, 3072, 3073, 4095, 4096, 4097, 6145, 8193]


def frame(ntx, nty, lengths, seed=0):
    """lengths[t] small Gaussians inside tile t, in shuffled order, every ninth
    with the depth of another of its tile; tile and depth of each."""
    import torch
    rng = np.random.default_rng(seed)
    W, Hh, f = 16 * ntx, 16 * nty, 400.0
    t = np.repeat(np.arange(ntx * nty), lengths)
    n = len(t)
    z = rng.uniform(2, 6, n).astype(np.float32)
    z[9::9] = np.where(t[9::9] == t[8:-1:9], z[8:-1:9], z[9::9])
    u, v = 16 * (t % ntx) + 7.5 + rng.uniform(-2, 2, n), 16 * (t // ntx) + 7.5 + rng.uniform(-2, 2, n)
    means = np.stack([(u - W / 2) / f * z, (v - Hh / 2) / f * z, z], 1)
    p = rng.permutation(n)
    g = (means[p], np.full((n, 3), 4e-4), np.tile([1.0, 0, 0, 0], (n, 1)), np.full(n, 0.02), np.full((n, 3), 0.5))
    g = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in g]
    pose = torch.tensor([1, 0, 0, 0, 0, 0, 0], dtype=torch.float32, device="cuda")
    return g, pose, gsr.make_camera(W, Hh, f, f, W / 2, Hh / 2, 0.2), t[p], z[p]


def check_lists(ntx, nty, lengths, seed=0):
    g, pose, cam, t, z = frame(ntx, nty, lengths, seed)
    st = gsr.render_fwd(*g, pose, cam)[3]
    K, ranges, ids = gsr.tile_lists(st, ntx * nty)
    st.release()
    assert K == len(t)
    ranges = ranges.cpu().numpy()
    np.testing.assert_array_equal(ranges[:, 1] - ranges[:, 0], lengths)
    np.testing.assert_array_equal(ids.cpu().numpy(), np.lexsort((np.arange(len(t)), z, t)))


@pytest.mark.parametrize("ntx,nty,base", [(4, 4, 20), (40, 32, 30), (75, 18, 30), (75, 18, 200), (75, 18, 700)])
def test_edges_of_runs_and_pieces(ntx, nty, base):
    """One workgroup per list up to 1,280 lists, one per four beyond; K below and
    above 2^18, by position and by length. The edges of the 1024-key network, of
    the 512-key runs, of the 2048-key pieces and of their merges, in
    neighbouring tiles."""
    lengths = np.random.default_rng(base).integers(0, 2 * base, ntx * nty)
    at = 0 if ntx * nty == 16 else 600
    lengths[at:at + len(EDGES)] = EDGES
    check_lists(ntx, nty, lengths, base)


def test_many_long_lists():
    """Every workgroup has several lists of more than 1,024 keys."""
    check_lists(75, 18, np.random.default_rng(1).integers(900, 2300, 75 * 18), 1)


def test_a_call_costs_the_same_whatever_its_context_served_before():
    """Lists of 300 keys, a few of 2000 among them: the tile lists' stage is not
    slower after a call with ten times the entries on the same state."""
    import torch
    lengths = np.full(75 * 43, 300)
    lengths[::250] = 2000
    g, pose, cam, _, _ = frame(75, 43, lengths)
    big = frame(75, 43, np.full(75 * 43, 1100))[:3]
    ctx = gsr.Context(0)

    def stage():
        got = []
        for _ in range(25):
            gsr.profile_enable(True, ctx)
            gsr.render_fwd(*g, pose, cam, ctx=ctx)[3].release()
            torch.cuda.synchronize()
            gsr.profile_enable(False, ctx)
            ms, calls = gsr.profile_read(ctx)["tile_bins"]
            got.append(ms / calls)
        return min(got)

    fresh = stage()
    gsr.render_fwd(*big[0], big[1], big[2], ctx=ctx)[3].release()
    after = stage()
    torch.cuda.synchronize()
    ctx.lib.gsr_ctx_destroy(ctypes.c_void_p(ctx.h.value) if hasattr(ctx.h, "value") else ctx.h)
    print(f"tile lists: {1e3 * fresh:.1f} us in a fresh context, {1e3 * after:.1f} us after a larger call")
    assert after < 1.2 * fresh


def test_many_short_lists_are_not_ordered():
    """65,536 tiles of four entries, just below and just above the 2^18 entries
    from which on the passes may go by length: the counting pass does not begin
    to make an order there (a third of its time), which would gain nothing."""
    import torch

    def stage(entries):
        lengths = np.full(256 * 256, 4)
        lengths[:abs(entries)] += np.sign(entries)
        g, pose, cam, _, _ = frame(256, 256, lengths)
        got = []
        for _ in range(15):
            gsr.profile_enable(True)
            gsr.render_fwd(*g, pose, cam)[3].release()
            torch.cuda.synchronize()
            gsr.profile_enable(False)
            ms, calls = gsr.profile_read()["bin_count"]
            got.append(ms / calls)
        return min(got)

    below, above = stage(-2000), stage(2000)
    print(f"counting: {1e3 * below:.1f} us below 2^18 entries, {1e3 * above:.1f} us above")
    assert above < 1.15 * below
