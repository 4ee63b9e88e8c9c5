"""The marched density of the SDF torus, at points known exactly, against its
distance evaluated in the marcher's own float32 steps: plain products under the
inner root, the outer sum fused.  The field is thin (width 1e-4), so that one
unit in the distance's last place moves the density by 1e-4 of itself.  The
network is zero.  Bound on the rest: the logit, at most 6, is a rounded
quotient (6 x 2^-24) in a sigmoid of a few units in the last place, as the
opacity's exponential: 2e-6 of the opacity."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu

F = np.float32
SIGMA, WIDTH = 0.1, 1e-4


def _points(n):
    """Points within 6 WIDTH of the surface, x on a grid of 2^-20 (so that an
    origin 3 before it is exact), and their float32 distance."""
    g = np.random.default_rng(41)
    th, ph = g.uniform(0, 2 * np.pi, (2, 4 * n))
    r = 0.2 + g.uniform(-5 * WIDTH, 5 * WIDTH, 4 * n)
    q = 0.5 + r * np.cos(ph)
    x = np.round(q * np.cos(th) * 2 ** 20) / 2 ** 20
    x, y, z = x.astype(F), (r * np.sin(ph)).astype(F), (q * np.sin(th)).astype(F)
    qx = np.sqrt(x * x + z * z) - F(0.5)
    assert qx.dtype == F
    # qx * qx is exact in float64, the sum then rounds to float32
    d = np.sqrt((qx.astype(np.float64) ** 2 + (y * y).astype(np.float64)).astype(F)) - F(0.2)
    near = np.flatnonzero(np.abs(d) < 6 * WIDTH)[:n]
    assert near.size == n
    return x[near], y[near], z[near], d[near]


@pytest.mark.parametrize("width,depth,enc_L", [(256, 8, 10), (64, 3, 6)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_marched_torus(width, depth, enc_L, dtype):
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    trunk = syn.normal_mlp(syn.rng(3, 42), [3 * (1 + 2 * enc_L)] + [width] * depth + [1])
    for w in trunk.W:
        w[:] = 0
    m = syn.Model(kind="mlp", bound=1.0, trunk=trunk, params=dict(enc_L=enc_L, sigma_mode="sdf", masked=False,
                                                                  sigma_max=SIGMA, width=WIDTH, sdf_shape=2))
    sc = gpu_scene([m], [syn.Instance(0, np.eye(3), np.zeros(3), 1.0)], dtype)
    x, y, z, dist = _points(2000)
    # one sample in the middle of [2, 4] along +x
    o = np.stack([x - F(3), y, z], axis=1)
    assert np.array_equal(o[:, 0] + F(3), x)
    d = np.tile(np.array([[1, 0, 0]], F), (x.size, 1))
    sigma = SIGMA / (1.0 + np.exp((dist / F(WIDTH)).astype(np.float64)))
    ref = -np.expm1(-2.0 * np.float64(F(SIGMA)) / SIGMA * sigma)
    for n in (100, x.size):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a[:n])).cuda()
        opac = api.march_depth(sc, api.array_rays(t(o), t(d)), n_samples=1, clip_to_bound=False, t_near=2.0,
                               t_far=4.0, dtype=dtype)[2]
        torch.cuda.synchronize()
        err = np.abs(opac.cpu().numpy().astype(np.float64) - ref[:n]) / ref[:n]
        log(f"[marched torus] {width} wide, {dtype}, {n} points: worst {err.max():.2e}, over: {int((err > 2e-6).sum())}")
        assert err.max() <= 2e-6
