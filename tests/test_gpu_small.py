"""Short lists run on the feature-split kernels, long ones on the
register-resident kernels: the same rays must give the same bits either way.
A ray array is evaluated alone (short lists) and repeated until its lists are
long; every copy has to match, at sizes around the 32-sample passes."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu


def _rays(n, seed):
    g = np.random.default_rng(seed)
    o = np.concatenate([g.uniform(-0.5, 0.5, (n, 2)), np.zeros((n, 1))], axis=1)
    t = np.concatenate([g.uniform(-1.0, 1.0, (n, 2)), np.full((n, 1), -6.0)], axis=1)
    d = (t - o) / np.linalg.norm(t - o, axis=1, keepdims=True)
    return o.astype(np.float32), d.astype(np.float32)


def _run(fn, o, d):
    import torch
    from paper_2308_04669_amd import api
    out = fn(api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()))
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


def _same_in_copies(fn, n, copies):
    o, d = _rays(n, 17 + n)
    one = _run(fn, o, d)
    many = _run(fn, np.tile(o, (copies, 1)), np.tile(d, (copies, 1)))
    for a, b in zip(one, many):
        assert np.array_equal(np.tile(a.view(np.uint32), copies), b.view(np.uint32))
    return one


@pytest.mark.parametrize("n", [1, 31, 32, 33, 257])
def test_short_and_long_lists_same_bits_infer(n):
    need_gpu()
    from paper_2308_04669_amd import api
    models, insts, _ = syn.sdf_scene(3, 6)
    nets = [syn.nedf_model(3, 200 + k, head_scale=4.0) for k in range(len(models))]
    sc = gpu_scene(models, insts, "bf16", nedf_models=nets)
    copies = -(-40000 // n)
    for refine in (0, 1, 3):
        dep, idn = _same_in_copies(lambda r: api.infer_depth_id(sc, r, dtype="bf16", refine_steps=refine), n, copies)
    log(f"[short lists] {n} rays, {copies} copies: {int((idn >= 0).sum())} hits")


@pytest.mark.parametrize("n,samples", [(1, 1), (3, 32), (5, 33), (40, 150)])
def test_short_and_long_lists_same_bits_march(n, samples):
    need_gpu()
    from paper_2308_04669_amd import api
    models, insts, _ = syn.sdf_scene(3, 6)
    sc = gpu_scene(models, insts, "bf16")
    dep, idn, opa = _same_in_copies(lambda r: api.march_depth(sc, r, n_samples=samples, dtype="bf16"), n, -(-4000 // n))
    log(f"[short lists] march {n} rays, {samples} samples: opacity up to {opa.max():.3f}")
