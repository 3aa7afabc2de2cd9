"""Rounding of the compositing backward's sums against 64 bits, on scenes whose
other steps are exact in 32 bits."""
import numpy as np
import pytest

from paper_2312_10070_amd import gsr

pytestmark = pytest.mark.gpu


def dev(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in arrays]


def eye():
    import torch
    return torch.tensor([1, 0, 0, 0, 0, 0, 0], dtype=torch.float32, device="cuda")


def rms(a):
    return float(np.sqrt((np.asarray(a) ** 2).mean()))


def test_moments_of_small_gaussians():
    """Lone Gaussians at the low-pass limit (variance 0.25 px^2, so the conic is
    exact) with centres on a grid of 2^-10 px, sums over pixels of q dx, q dy,
    q dx^2, q dy^2 read back from the gradients of means and scales (factors
    that are powers of two).

    A pixel's term has about eight roundings (exponent 2, exponential 2, opacity,
    transmittance 2, moment 2) of at most 2^-24, rms 2^-24 / sqrt(3), and some six pixels
    carry a sum, which adds as many: below 3 * 2^-24 together, rms over the Gaussians."""
    import torch
    rng = np.random.default_rng(0)
    f, s = 64.0, 2.0 ** -24
    gx, gy = np.meshgrid(np.arange(1, 31), np.arange(1, 31))
    n = gx.size
    u = 16.0 * gx.ravel() + rng.integers(0, 8192, n) / 1024.0
    v = 16.0 * gy.ravel() + rng.integers(0, 8192, n) / 1024.0
    o = rng.uniform(0.1, 0.9, n).astype(np.float32)
    means = np.stack([(u - 256) / f, (v - 256) / f, np.ones(n)], 1)
    g = dev(means, np.full((n, 3), s), np.tile([1.0, 0, 0, 0], (n, 1)), o, np.tile([1.0, 0, 0], (n, 1)))
    assert np.array_equal(g[0].double().cpu().numpy(), means)
    st = gsr.render_fwd(*g, eye(), gsr.make_camera(512, 512, f, f, 256.0, 256.0, 0.2), gsr.RasterOpts(lowpass=0.25))[3]
    gC = torch.zeros((3, 512, 512), device="cuda")
    gC[0] = 1.0
    out = gsr.render_bwd(st, gC, torch.zeros((512, 512), device="cuda"))
    torch.cuda.synchronize()
    st.release()
    out = {k: x.double().cpu().numpy() for k, x in out.items()}
    p = 4.0 * np.float64(np.float32(-0.5) * np.float32(1.4426950408889634))
    dx = np.floor(u)[:, None] + np.arange(-6, 8) - u[:, None]
    dy = np.floor(v)[:, None] + np.arange(-6, 8) - v[:, None]
    X, Y = dx[:, None, :], dy[:, :, None]
    q = o.astype(np.float64)[:, None, None] * 2.0 ** (p * (X * X + Y * Y))
    q[q < np.float32(1.0 / 255.0)] = 0.0
    moment = f * 4.0
    second = f * f * 16.0 * s
    for name, got, w in (("dx", out["means"][:, 0] / moment, X), ("dy", out["means"][:, 1] / moment, Y),
                         ("dx^2", out["scales"][:, 0] / second, X * X), ("dy^2", out["scales"][:, 1] / second, Y * Y)):
        err = (got - (q * w).sum((1, 2))) / (q * np.abs(w)).sum((1, 2))
        print(f"sum of q {name}: rms {rms(err):.2e}, largest {np.abs(err).max():.2e}")
        assert rms(err) <= 3 * 2.0 ** -24, name


def test_opacities_below_an_alpha_gradient():
    """200 layers that fill the image, alpha of each its opacity exactly, with an
    upstream gradient of alpha a thousand times that of colour: the term of what
    lies behind a layer is small beside the alpha term, and is not to be rounded
    to its size at every layer.

    The alpha term takes a difference, a reciprocal (1 ulp, twice a rounding), a
    product, a sum, and the opacity factor: below 2 * 2^-24, rms over layers."""
    import torch
    errs = []
    for seed in range(10):
        rng = np.random.default_rng(seed)
        n, W = 200, 16
        o = rng.integers(270, 400, n) / 65536.0  # (1 - o exact)
        col = np.zeros((n, 3))
        col[:, 0] = rng.uniform(0.5, 1, n).astype(np.float32)
        z = 1 + 0.001 * np.arange(n)
        g = dev(np.stack([0 * z, 0 * z, z], 1), np.full((n, 3), 1e6), np.tile([1.0, 0, 0, 0], (n, 1)), o, col)
        cam = gsr.make_camera(W, W, 64.0, 64.0, 8.0, 8.0, 0.2, (0.0, 0.0, 1.0))
        color, _, _, st = gsr.render_fwd(*g, eye(), cam)
        T = float(color[2, 3, 3])  # the final transmittance: the third channel is background alone
        assert bool((color[2] == T).all()) and 0.3 < T < 0.5
        w = float(np.float32(1e-3))
        gC = torch.zeros_like(color)
        gC[0] = w
        out = gsr.render_bwd(st, gC, torch.zeros((W, W), device="cuda"), torch.ones((W, W), device="cuda"))
        got = out["opacities"].double().cpu().numpy() / (W * W)
        st.release()
        want, behind, t = np.empty(n), 0.0, T
        for j in range(n - 1, -1, -1):
            t /= 1 - o[j]
            want[j] = t * w * col[j, 0] - (behind - T) / (1 - o[j])
            behind += w * col[j, 0] * o[j] * t
        errs.append((got - want) / want)
    err = np.concatenate(errs)
    print(f"dL/do: rms {rms(err):.2e}, largest {np.abs(err).max():.2e}")
    assert rms(err) <= 2 * 2.0 ** -24


def test_opacity_gradient_is_the_sum_itself():
    """One Gaussian that fills the image at alpha = o = 3/4, an upstream gradient
    of alpha alone: T, its reciprocal and the per-pixel gradients are exact, 256
    equal ones add up exactly, and so dL/do = 256 ga, with no rounding at all."""
    import torch
    W = 16
    g = dev([[0, 0, 1]], np.full((1, 3), 1e6), [[1.0, 0, 0, 0]], [0.75], np.zeros((1, 3)))
    cam = gsr.make_camera(W, W, 64.0, 64.0, 8.0, 8.0, 0.2)
    _, _, _, st = gsr.render_fwd(*g, eye(), cam)
    zero = torch.zeros((W, W), device="cuda")
    for ga in np.random.default_rng(0).uniform(1, 2, 64).astype(np.float32):
        out = gsr.render_bwd(st, torch.zeros((3, W, W), device="cuda"), zero, torch.full((W, W), float(ga), device="cuda"))
        assert float(out["opacities"][0]) == 256 * float(ga)
    st.release()
