"""The matrix-core training kernel (csrc/train_mfma.h) against the FP64 oracle at the shapes it has
besides the three-layer ones (width 16, 1 and 4 hidden layers, learned frames), at batches around
its 16-sample tiles, of fewer tiles than workgroups and of several tiles per wave pair.

Tolerance: the norm bound of the training parity tests, 1e-3 (a hidden unit within rounding of its
ReLU's kink moves one sample's share of a gradient, at most a few of these batches' samples).
"""
import numpy as np
import pytest

import oracle
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


def _close(g, ref, what):
    ref = np.asarray(ref, np.float64).ravel()
    assert np.linalg.norm(g.ravel() - ref) <= 1e-3 * np.linalg.norm(ref), what


@pytest.mark.parametrize("C,H,NH,nf,albedo", [(8, 16, 2, 0, False), (16, 16, 4, 0, True), (8, 64, 1, 0, True),
                                              (16, 32, 4, 0, False), (16, 64, 3, 0, True), (8, 64, 3, 2, False),
                                              (16, 64, 2, 1, False), (16, 32, 3, 2, False)])
@pytest.mark.parametrize("n", [1, 15, 17, 1029, 20011])
def test_gradients_at_tile_edges(nam, torch, C, H, NH, nf, albedo, n):
    ctx = nam.Context(0)
    r = wl.rngs(81)
    m = wl.make_material(r[0], r[1], 32, 16, C, 5, [H] * NH, n_frames=nf, albedo=albedo,
                         address=wl.CLAMP if n == 17 else wl.WRAP)
    m.params = (m.params + 0.05 * r[1].standard_normal(m.params.size)).astype(np.float32)
    q = wl.uniform_queries(r[2], n, -0.5, 4.5)
    tgt = r[3].random((n, m.dims[-1])).astype(np.float32)
    if n > 1000:
        q.uv[3, 0] = np.nan                              # contributes nothing
    model = nam.Model.from_workload(ctx, m)
    params = np.concatenate([m.frame_params, m.params]) if nf else m.params
    tex, par, tg = (torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
                    for a in (nam.concat_levels(m.levels), params, tgt))
    d = nam.to_device(q)
    loss, d_tex, d_par = model.loss_backward(tex, par, *d, tg)
    if nf:
        L, dP, dF, dL = oracle.loss_grad_frames(m.levels, m.dims, m.params, m.frame_params, nf, q.uv, q.lod, q.wi,
                                                q.wo, tgt, m.address)
        dP = np.concatenate([dF, dP])
    else:
        L, dP, dL = oracle.loss_grad(m.levels, m.dims, m.params, q.uv, q.lod, q.wi, q.wo, tgt, m.address)
    assert abs(loss.item() - L) <= 1e-5 * L
    _close(d_par.cpu().numpy(), dP, "parameters")
    _close(d_tex.cpu().numpy(), nam.concat_levels(dL), "texels")
    # parameter gradients do not depend on scheduling; a given output gradient gives the same ones
    assert torch.equal(model.loss_backward(tex, par, *d, tg)[2], d_par)
    rgb = model.forward(tex, par, *d)
    keep = torch.isfinite(d[0]).all(1, keepdim=True)
    assert torch.isnan(rgb[~keep[:, 0]]).all()
    d_rgb = torch.where(keep, 2.0 / (3.0 * n) * (torch.nan_to_num(rgb) - tg), torch.zeros_like(tg))
    _close(model.backward(tex, par, *d, d_rgb)[1].cpu().numpy(), dP, "parameters from output gradients")
