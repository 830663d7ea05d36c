"""The encoder's codes and parameter gradient on the matrix cores (csrc/encoder.hip) against the FP64
oracle at batches around its 16-sample tiles, of fewer tiles than waves and of several tiles per wave, at the
smallest and largest shapes.

Tolerances: codes within 1e-5 relative to max(1, |z|) (FP32 roundings through at most three layers);
gradients norm-relative 1e-3 (a hidden unit within rounding of its ReLU's kink moves one sample's
share of a gradient, at most a few of these batches' samples).
"""
import numpy as np
import pytest

import oracle
from paper_2305_02678_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A,C,HE,NHE", [(4, 8, 16, 1), (4, 16, 32, 2), (8, 8, 16, 2), (16, 16, 64, 2), (8, 16, 64, 1)])
@pytest.mark.parametrize("n", [1, 15, 17, 65, 4103, 70001])
def test_gradients_at_tile_edges(A, C, HE, NHE, n):
    import torch
    from paper_2305_02678_amd import nam
    rng = np.random.default_rng(71)
    M, size = 4, 16
    attr = [rng.random((size >> l, size >> l, A)).astype(np.float32) for l in range(M)]
    dims, ep = wl.encoder_params(rng, A, C, [HE] * NHE)
    ep = (ep + 0.05 * rng.standard_normal(ep.size)).astype(np.float32)
    q = wl.uniform_queries(rng, n, -0.5, M - 0.5)
    dz = rng.standard_normal((n, C)).astype(np.float32)
    if n > 1:
        q.uv[n - 2, 1] = np.nan                          # contributes nothing
    enc = nam.Encoder(nam.Context(0), dims, size, size, M, wl.WRAP)
    args = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
            for a in (ep, np.concatenate([l.reshape(-1, A) for l in attr]), q.uv, q.lod, dz)]
    z = enc.encode_queries(*args[:4]).cpu().numpy().astype(np.float64)
    exact = oracle.encode_queries(attr, dims, ep, q.uv, q.lod, wl.WRAP)
    ok = np.isfinite(exact).all(1)
    assert np.isnan(z[~ok]).all() and (~ok).sum() == (n > 1)
    assert (np.abs(z[ok] - exact[ok]) <= 1e-5 * np.maximum(1.0, np.abs(exact[ok]))).all()
    g = enc.backward(*args)
    ref = np.asarray(oracle.encoder_backward(attr, dims, ep, q.uv, q.lod, dz, wl.WRAP), np.float64).ravel()
    assert np.linalg.norm(g.cpu().numpy().ravel() - ref) <= 1e-3 * np.linalg.norm(ref)
    assert torch.equal(enc.backward(*args), g)           # independent of scheduling
