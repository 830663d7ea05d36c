"""Training on pyramids of 2^31 values, which the matrix-core kernels' 32-bit offsets do not reach and
the vector kernels (csrc/train_vec.h) take: every family of shapes against the same call on a small
pyramid that holds the texels the samples meet.  Samples lie on texel centres of level 0 (uv exact in
FP32), so both calls see the same codes; the two kernels' FP32 sums are held to 1e-5 of their norm."""
import numpy as np
import pytest

from paper_2305_02678_amd import workloads as wl

pytestmark = pytest.mark.gpu

W, H = 16384, 8192                             # x 16 channels: 2^31 values


@pytest.mark.parametrize("hidden,nf,outputs", [([64] * 3, 0, 3), ([32] * 2, 0, 6), ([16], 0, 3), ([64] * 3, 2, 3), ([32] * 2, 1, 3)])
def test_pyramid_of_2_31_values(hidden, nf, outputs):
    import torch
    from paper_2305_02678_amd import nam
    ctx = nam.Context(0)
    C, n, side = 16, 500, 32
    r = wl.rngs(110)
    m = wl.make_material(r[0], r[1], side, side, C, 1, hidden, n_frames=nf, albedo=outputs == 6)
    params = np.concatenate([m.frame_params, m.params]) if nf else m.params
    params = torch.from_numpy((params + 0.05 * r[1].standard_normal(params.size)).astype(np.float32)).cuda()
    at = r[2].integers(0, side, (n, 2))                                   # in the small texture
    far = np.stack([r[3].choice(W, side, replace=False), r[3].choice(H, side, replace=False)], 1)
    far[0], far[1] = (0, 0), (W - 1, H - 1)
    big_at = np.stack([far[at[:, 0], 0], far[at[:, 1], 1]], 1)
    q = wl.uniform_queries(r[2], n, 0.0, 0.0)
    small_tex = torch.from_numpy(np.ascontiguousarray(nam.concat_levels(m.levels), np.float32)).cuda()
    index = torch.from_numpy(far[:, 1][:, None] * W + far[:, 0][None, :]).reshape(-1).cuda()   # [y][x]
    big_tex = torch.zeros(W * H, C, device="cuda")
    big_tex[index] = small_tex
    target = torch.rand(n, outputs, generator=torch.Generator().manual_seed(111)).cuda()
    d_rgb = torch.randn(n, outputs, generator=torch.Generator().manual_seed(112)).cuda()
    got = []
    for tex, w, h, where in ((small_tex, side, side, at), (big_tex, W, H, big_at)):
        model = nam.Model(ctx, w, h, C, 1, m.dims, m.address, nf)
        q.uv[:] = (where + 0.5) / np.array([w, h])
        d = nam.to_device(q)
        rgb = model.forward(tex, params, *d)
        loss, d_tex, d_par = model.loss_backward(tex, params, *d, target)
        g_tex, g_par = model.backward(tex, params, *d, d_rgb)
        if w == W:
            assert int(d_tex.count_nonzero(1).count_nonzero()) <= n
            d_tex, g_tex = d_tex[index], g_tex[index]
        got.append((rgb, loss, d_tex, d_par, g_tex, g_par))
        torch.cuda.synchronize()
    for a, b in zip(*got):
        assert float((a - b).norm()) <= 1e-5 * float(a.norm())
