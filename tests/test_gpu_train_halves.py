"""The training kernel's products in FP16 halves (csrc/train_mfma.h) against FP64 autograd: samples
whose gradients differ by many powers of two in one tile (each has its own scale), and sums over many
samples of either sign (a rounding that leans to one side would add up in them; with given output
gradients, as the FP32 softplus of a loss leans by itself).

Samples with a hidden unit within 1e-5 of its kink are left out (a NaN code or query contributes
nothing), so that every ReLU is on the same side in FP64.  Tolerances: a pair of halves holds 22 bits of
a sample's largest value, so each of the at most nine products in a row is within 2^-21 of it times the
root of 64 terms at worst, 3e-5 together, for one sample's gradient; sums over samples of independent
errors of 2^-24 stay within 1e-6 of their norm, where a bias of 1/5 of that would reach 3e-6 at 65,536.
A sample far above the others takes no bits from the gradients that it does not touch itself: these are
held to the bound of one sample's gradient on their own norm, row by row.
"""
import numpy as np
import pytest

from paper_2305_02678_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def nam(torch):
    from paper_2305_02678_amd import nam as n
    n.lib()
    return n


def _case(torch, nam, C, hidden, n, seed):
    """Model, queries and their codes, which samples are not near a kink, and the FP64 network."""
    r = wl.rngs(seed)
    m = wl.make_material(r[0], r[1], 16, 16, C, 3, hidden)
    m.params = (m.params + 0.05 * r[1].standard_normal(m.params.size)).astype(np.float32)
    q = wl.uniform_queries(r[2], n, 0.0, 1.0)
    at = r[3].integers(0, 16, (n, 2))                    # a texel of level 0 and its centre
    z = torch.from_numpy(np.ascontiguousarray(m.levels[0], np.float32)[at[:, 1], at[:, 0]])
    q.uv[:], q.lod[:] = (at + 0.5) / 16, 0.0
    p64 = torch.from_numpy(m.params).double().requires_grad_()

    def net(zz):
        x, o, margin = torch.cat([zz, torch.from_numpy(q.wi).double(), torch.from_numpy(q.wo).double()], 1), 0, None
        for k, (a, b) in enumerate(zip(m.dims[:-1], m.dims[1:])):
            y = x @ p64[o:o + a * b].view(b, a).T + p64[o + a * b:o + a * b + b]
            o += a * b + b
            if k < len(m.dims) - 2:
                near = (y.abs().min(1).values / y.abs().max(1).values).detach()
                margin = near if margin is None else torch.minimum(margin, near)
                x = y.relu()
        return torch.nn.functional.softplus(y), margin

    keep = net(z.double())[1] > 1e-5
    assert keep.float().mean() > 0.9
    model = nam.Model.from_workload(nam.Context(0), m)
    tex, par = (torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (nam.concat_levels(m.levels), m.params))
    return model, tex, par, q, z, keep, net, p64


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2), (8, [64])])
def test_samples_of_different_scale(nam, torch, C, hidden):
    n = 333
    model, _, par, q, z, keep, net, p64 = _case(torch, nam, C, hidden, n, 91)
    k = torch.from_numpy(np.random.default_rng(92).integers(0, 60, (n, 1)))
    target = (-torch.exp2(k.double())).float().expand(n, 3).contiguous()
    zz = z.double().requires_grad_()
    e = torch.where(keep[:, None], net(zz)[0] - target.double(), 0.0)
    dz, dp = torch.autograd.grad((e ** 2).sum() / e.numel(), (zz, p64))
    z[~keep] = float("nan")
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    _, gz, gp = model.loss_backward_codes(par, *dev, target.cuda())
    gz = gz.cpu().double()
    assert (gz[~keep] == 0).all()
    err = ((gz - dz).norm(dim=1) / dz.norm(dim=1))[keep]
    assert err.max() <= 3e-5
    assert (gp.cpu().double() - dp).norm() <= 3e-5 * dp.norm()


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2)])
def test_sums_over_either_sign(nam, torch, C, hidden):
    n = 65536
    model, tex, par, q, z, keep, net, p64 = _case(torch, nam, C, hidden, n, 93)
    d_rgb = torch.from_numpy(np.random.default_rng(94).standard_normal((n, 3)).astype(np.float32))
    dp, = torch.autograd.grad((net(z.double())[0] * torch.where(keep[:, None], d_rgb.double(), 0.0)).sum(), p64)
    q.uv[~keep.numpy()] = np.nan
    gp = model.backward(tex, par, *nam.to_device(q), d_rgb.cuda())[1]
    assert (gp.cpu().double() - dp).norm() <= 1e-6 * dp.norm()


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2), (8, [64])])
@pytest.mark.parametrize("n", [16, 65536])
@pytest.mark.parametrize("above", [10, 16, 24, 30, 50, 70])
def test_small_samples_beside_large_ones(nam, torch, C, hidden, n, above):
    """Output gradients of order 1, but for one sample of a tile (n = 16), or one of the first tile of
    every wave: 2^above, in the first output alone."""
    model, tex, par, q, z, keep, net, p64 = _case(torch, nam, C, hidden, n, 95)
    d_rgb = torch.from_numpy(np.random.default_rng(96).standard_normal((n, 3)).astype(np.float32))
    large = torch.zeros(n, dtype=torch.bool)
    large[3:16 * 1024:16] = True                         # at most 256 CUs of 4 pairs of waves
    d_rgb[large] = torch.tensor([2.0 ** above, 0.0, 0.0])
    dp, = torch.autograd.grad((net(z.double())[0] * torch.where(keep[:, None], d_rgb.double(), 0.0)).sum(), p64, retain_graph=True)
    q.uv[~keep.numpy()] = np.nan
    gp = model.backward(tex, par, *nam.to_device(q), d_rgb.cuda())[1].cpu().double()
    # what the large samples touch: their share of the gradient is not zero
    share, = torch.autograd.grad((net(z.double())[0] * torch.where((keep & large)[:, None], d_rgb.double(), 0.0)).sum(), p64)
    o, rows = 0, 0
    dims = [C + 6] + hidden + [3]
    for a, b in zip(dims[:-1], dims[1:]):
        for r in range(b):
            row = torch.cat([torch.arange(o + r * a, o + (r + 1) * a), torch.tensor([o + a * b + r])])
            if (share[row] == 0).all() and (dp[row] != 0).any():
                rows += 1
                assert (gp[row] - dp[row]).norm() <= 3e-5 * dp[row].norm(), (a, b, r)
        o += a * b + b
    assert rows >= (2 if n > 16 else 10)


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2)])
def test_units_without_weights(nam, torch, C, hidden):
    """A unit of every layer whose weights and bias are zero: no gradient through it, and the time of a
    decoder without such units (no FP32 repeat of every tile's forward pass)."""
    n = 1 << 18
    model, _, par, q, z, _, _, _ = _case(torch, nam, C, hidden, n, 97)
    unit, o, dims = [], 0, [C + 6] + hidden + [3]
    for a, b in zip(dims[:-2], dims[1:-1]):
        unit += [*range(o + 5 * a, o + 6 * a), o + a * b + 5]
        o += a * b + b
    small = par.clone()
    small[unit] = 0.0
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    target = torch.rand(n, 3, device="cuda")
    times = []
    for p in (par, small):
        t = []
        for _ in range(15):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            grad = model.loss_backward_codes(p, *dev, target)[2]
            e[1].record()
            torch.cuda.synchronize()
            t.append(e[0].elapsed_time(e[1]))
        times.append(sorted(t)[len(t) // 2])
    print(f"{times[0]:.3f} ms, with units without weights {times[1]:.3f} ms", flush=True)
    assert (grad[unit] == 0).all()
    assert times[1] <= 1.15 * times[0]


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2)])
def test_infinite_weight_of_an_inactive_unit(nam, torch, C, hidden):
    """A weight of minus infinity on a direction that is always positive turns its unit off and leaves
    loss and gradients finite: the same gradients as without the unit."""
    n = 1000
    model, _, par, q, z, _, _, _ = _case(torch, nam, C, hidden, n, 99)
    a = C + 6
    q.wo[:] = np.abs(q.wo) + np.float32(0.01)
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    target = torch.rand(n, 3, device="cuda")
    off = par.clone()
    off[5 * a:6 * a] = 0.0
    off[5 * a + C + 5] = float("-inf")
    without = par.clone()
    without[5 * a:6 * a] = 0.0
    without[a * hidden[0] + 5] = -1.0
    loss, dz, dp = model.loss_backward_codes(off, *dev, target)
    loss1, dz1, dp1 = model.loss_backward_codes(without, *dev, target)
    assert abs(float(loss) - float(loss1)) <= 1e-6 * float(loss1)
    assert torch.isfinite(dz).all() and torch.isfinite(dp).all()
    assert (dz - dz1).norm() <= 1e-6 * dz1.norm() and (dp - dp1).norm() <= 1e-6 * dp1.norm()


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2)])
@pytest.mark.parametrize("k", [118, 60, -60, -110])
def test_layers_of_any_scale(nam, torch, C, hidden, k):
    """The first layer times 2^k and the second layer's weights times 2^-k, which changes no output: every
    layer's gradients and the codes' against FP64."""
    n = 333
    model, _, par, q, z, keep, net, p64 = _case(torch, nam, C, hidden, n, 101)
    dims, o, layers = [C + 6] + hidden + [3], 0, []
    for a, b in zip(dims[:-1], dims[1:]):
        layers.append((o, o + a * b, o + a * b + b))
        o += a * b + b
    with torch.no_grad():
        p64[layers[0][0]:layers[0][2]] *= 2.0 ** k
        p64[layers[1][0]:layers[1][1]] *= 2.0 ** -k
    par.copy_(p64.detach().float())
    target = torch.rand(n, 3, generator=torch.Generator().manual_seed(102))
    zz = z.double().requires_grad_()
    e = torch.where(keep[:, None], net(zz)[0] - target.double(), 0.0)
    dz, dp = torch.autograd.grad((e ** 2).sum() / e.numel(), (zz, p64))
    z[~keep] = float("nan")
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    _, gz, gp = model.loss_backward_codes(par, *dev, target.cuda())
    gz, gp = gz.cpu().double(), gp.cpu().double()
    assert (gz - dz).norm() <= 3e-5 * dz.norm()
    for first, _, last in layers:
        assert (gp[first:last] - dp[first:last]).norm() <= 3e-5 * dp[first:last].norm()


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [32] * 2), (16, [16] * 2)])
@pytest.mark.parametrize("k", [12, 20])
def test_small_weights_beside_a_large_one(nam, torch, C, hidden, k):
    """One weight 2^k times the others of its layer, on a channel that is always zero: the loss and every
    gradient but that channel's are those of the other weights."""
    n = 333
    model, _, par, q, z, _, _, p64 = _case(torch, nam, C, hidden, n, 103)
    z[:, 0] = 0.0
    with torch.no_grad():
        p64[3 * (C + 6)] = 2.0 ** k
    par.copy_(p64.detach().float())
    zz, o = z.double().requires_grad_(), 0
    x = torch.cat([zz, torch.from_numpy(q.wi).double(), torch.from_numpy(q.wo).double()], 1)
    keep = torch.ones(n, dtype=torch.bool)
    dims = [C + 6] + hidden + [3]
    for i, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        y = x @ p64[o:o + a * b].view(b, a).T + p64[o + a * b:o + a * b + b]
        o += a * b + b
        keep &= (y.abs().min(1).values > 1e-5 * y.abs().max(1).values) if i < len(hidden) else True
        x = y.relu()
    target = torch.rand(n, 3, generator=torch.Generator().manual_seed(104))
    e = torch.where(keep[:, None], torch.nn.functional.softplus(y) - target.double(), 0.0)
    dz, dp = torch.autograd.grad((e ** 2).sum() / e.numel(), (zz, p64))
    z[~keep] = float("nan")
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    _, gz, gp = model.loss_backward_codes(par, *dev, target.cuda())
    assert (gz.cpu().double() - dz)[:, 1:].norm() <= 3e-5 * dz[:, 1:].norm()
    assert (gp.cpu().double() - dp).norm() <= 3e-5 * dp.norm()


@pytest.mark.parametrize("C,hidden", [(16, [64] * 3), (8, [64] * 2), (16, [64]), (16, [32] * 3), (8, [16] * 2)])
def test_sum_of_the_codes_gradients(nam, torch, C, hidden):
    """Gradients of one sign, summed over 65,536 samples: what a rounding does alike to every sample (of a
    weight, above all) stays in the sum, the rest averages out.  One rounding, 2^-24, is left for the
    loss's factor and the softplus."""
    n = 65536
    model, _, par, q, z, keep, net, _ = _case(torch, nam, C, hidden, n, 200)
    target = torch.full((n, 3), -100.0)
    zz = z.double().requires_grad_()
    e = torch.where(keep[:, None], net(zz)[0] - target.double(), 0.0)
    total = torch.autograd.grad((e ** 2).sum() / e.numel(), zz)[0].sum(0)
    z[~keep] = float("nan")
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (z.numpy(), q.wi, q.wo)]
    got = model.loss_backward_codes(par, *dev, target.cuda())[1].cpu().double().sum(0)
    assert (got - total).norm() <= 2.0 ** -24 * total.norm()


@pytest.mark.parametrize("C,hidden", [(16, [64]), (8, [32]), (16, [16])])
def test_last_bit_of_output_gradients(nam, torch, C, hidden):
    """Output gradients whose last bit is in neither half: each code's gradient is one product, held to
    2^-24 in the norm over the samples (leaving the bit out would cost 2^-23 of every one)."""
    H, n = hidden[0], 64 * 64
    r = wl.rngs(211)
    m = wl.make_material(r[0], r[1], 64, 64, C, 3, hidden)
    W1, b1, W2, b2 = np.zeros((H, C + 6)), np.zeros(H), np.zeros((3, H)), np.full(3, 40.0)     # logistic(q) = 1
    W1[:8, :8], b1[:8], W2[0, :8] = np.eye(8), 1.0, 31 / 16
    params = np.concatenate([v.ravel() for v in (W1, b1, W2, b2)]).astype(np.float32)
    q = wl.uniform_queries(r[2], n, 0.0, 1.0)
    at = np.stack([np.arange(n) % 64, np.arange(n) // 64], 1)         # every sample on a texel of its own
    q.uv[:], q.lod[:] = (at + 0.5) / 64, 0.0
    low = (2 * r[3].integers(1024, 2047, n) + 1) * 2.0 ** -23
    d_rgb = np.zeros((n, 3), np.float32)
    d_rgb[:, 0] = 1.0 + r[3].integers(0, 31, n) * 2.0 ** -10 + low * r[3].choice([-1.0, 1.0], n)
    model = nam.Model.from_workload(nam.Context(0), m)
    tex = torch.zeros(nam.concat_levels(m.levels).shape, device="cuda")
    dev = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (q.uv, q.lod, q.wi, q.wo, d_rgb)]
    got = model.backward(tex, torch.from_numpy(params).cuda(), *dev)[0][:n, :8].cpu().double()
    want = torch.from_numpy(d_rgb[:, :1].astype(np.float64) * (31 / 16)).expand(n, 8)
    assert (got - want).norm() <= 2.0 ** -24 * want.norm()
