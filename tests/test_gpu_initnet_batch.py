"""The initialiser's kernels over batch sizes: the forward and data-gradient
kernels for few and for many pixels give a sample the same bits, the weight
and bias gradients of a batch are the sum of its samples', and packing at every
pooling factor that has its own code."""
import numpy as np
import pytest

from paper_2312_10070_amd import gsr, initnet

pytestmark = pytest.mark.gpu

SHAPES = [(120, 160, 8), (60, 80, 64), (30, 40, 64), (15, 20, 64), (8, 10, 64)]


def run(net, x, dout):
    import torch
    b = x.shape[0]
    net.set_input(x)
    out = net.forward(b)
    net.backward(b, dL_dout=dout)
    _, g = net.get_params(with_grads=True)
    acts = [net.activation(l, b, SHAPES[l]) for l in range(1, 5)]
    torch.cuda.synchronize()
    return out, g, acts


@pytest.mark.parametrize("batch", [1, 2, 5, 6, 21])  # 5 / 6 and 20 / 21 samples: either side of the few-pixel kernel's limit
def test_batch_equals_its_samples(batch):
    import torch
    net = gsr.InitNet(max_batch=21)
    rng = np.random.default_rng(batch)
    flat = initnet.init_params(3)
    lay, _ = initnet.layout()
    for name, shape, off in lay:
        if name.startswith("b"):
            flat[off:off + shape[0]] = rng.normal(0, 0.05, shape[0])
    net.set_params(torch.from_numpy(flat).cuda())
    x = torch.from_numpy(rng.uniform(0, 1, (batch, 120, 160, 8)).astype(np.float32)).cuda().bfloat16()
    dout = torch.from_numpy(rng.normal(size=(batch, 6)).astype(np.float32)).cuda()
    out, g, acts = run(net, x, dout)
    total, size = torch.zeros_like(g, dtype=torch.float64), torch.zeros_like(g, dtype=torch.float64)
    for i in range(batch):
        o1, g1, a1 = run(net, x[i:i + 1].contiguous(), dout[i:i + 1].contiguous())
        assert torch.equal(o1[0], out[i])
        for (a, d), (b, e) in zip(acts, a1):
            assert torch.equal(a[i], b[0]) and torch.equal(d[i], e[0])
        total += g1.double()
        size += g1.double().abs()
    # the same products added in another order, in FP32: a sample's sums carry up to ~1e-6 of their largest terms,
    # which are of the order of the parameter group's largest gradient
    for name, shape, off in lay:
        sl = slice(off, off + int(np.prod(shape)))
        err = (g[sl].double() - total[sl]).abs().max().item()
        assert err <= 2e-5 * size[sl].max().item(), (name, err, size[sl].max().item())


@pytest.mark.parametrize("f", [1, 2, 3, 4, 5])
def test_pack_every_factor(f):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(f)
    h, w = 120 * f, 160 * f
    rc, oc = (torch.rand((3, h, w), device="cuda", generator=gen) for _ in range(2))
    rd, od = (1 + 3 * torch.rand((h, w), device="cuda", generator=gen) for _ in range(2))
    dst = torch.empty((120, 160, 8), device="cuda", dtype=torch.bfloat16)
    gsr.pack_rgbd_pair(rc, rd, oc, od, dst, 0.25)
    r, o = torch.cat([rc, 0.25 * rd[None]]).double(), torch.cat([oc, 0.25 * od[None]]).double()
    ref = torch.nn.functional.avg_pool2d(torch.cat([r, 4 * (o - r)])[None], f)[0].permute(1, 2, 0)
    # BF16 keeps 8 bits; the FP32 sums of up to 25 values below 8 add 25 ulps of 8 at most
    assert ((dst.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 25 * 2.0 ** -21).all()
