"""The secant refinement starts from the same seeds in every kernel: pixels of
instances whose half bracket width is the rounding-critical kind (the rounded
product and the fused one give neighbouring upper seeds) refine to the same
bits in short lists and in long ones."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu

H = 0.05


def _critical_scales(n):
    """Scales whose seed D + H s rounds differently when the product is
    rounded first, for every other depth D in [4, 8) (the rounded product is
    then half a unit in D's last place, the exact one is not)."""
    s = np.random.default_rng(9).uniform(0.7, 1.3, 20000).astype(np.float32)[:, None]
    h = np.float32(H)
    D = (5.5 + np.arange(64) * 2.0 ** -21).astype(np.float32)
    rounded = D + h * s
    fused = (D.astype(np.float64) + np.float64(h) * s.astype(np.float64)).astype(np.float32)
    ok = s[(rounded != fused).sum(1) >= 24, 0]
    assert ok.size >= n
    return [float(x) for x in ok[:n]]


def test_refinement_same_bits_in_short_and_long_lists():
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    model = syn.nerf_model(3, 150, sigma_mode="sdf", sdf_shape=0)
    net = syn.nedf_model(3, 200)
    scales = _critical_scales(6)
    insts = [syn.Instance(0, np.eye(3), np.array([4.0 * k, 0.0, -6.0]), s) for k, s in enumerate(scales)]
    sc = gpu_scene([model], insts, "bf16", nedf_models=[net])
    g = np.random.default_rng(4)
    n = 40 * len(insts)
    o = np.zeros((n, 3), np.float32)
    o[:, 0] = np.repeat([4.0 * k for k in range(len(insts))], 40) + g.uniform(-0.3, 0.3, n)
    o[:, 1] = g.uniform(-0.3, 0.3, n)
    d = np.tile(np.float32([0.0, 0.0, -1.0]), (n, 1))
    limit = 3 * torch.cuda.get_device_properties(0).multi_processor_count * 32  # pixels of the short lists' kernel
    copies = -(-2 * limit // n)

    def run(o, d):
        ws = api.Workspace()
        rays = api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
        # p_lo = 0, p_hi = 1: every pair is marched, so that every ray through an object has a hit
        dep, idn = api.infer_depth_id(sc, rays, dtype="bf16", p_lo=0.0, p_hi=1.0, refine_steps=1, refine_h=H, ws=ws)
        torch.cuda.synchronize()
        return dep.cpu().numpy().view(np.uint32), idn.cpu().numpy(), api.ws_counters(ws)["pairs"]

    d1, i1, p1 = run(o, d)
    dn, idn, pn = run(np.tile(o, (copies, 1)), np.tile(d, (copies, 1)))
    log(f"[refine bits] {p1} and {pn} refined pixels, depths {d1.view(np.float32).min():.2f} .. "
        f"{d1.view(np.float32)[i1 >= 0].max():.2f}, {int((np.tile(d1, copies) != dn).sum()) // copies} pixels differ")
    assert n // 2 < p1 <= limit - 32 and pn > limit
    assert np.array_equal(np.tile(i1, copies), idn)
    assert np.array_equal(np.tile(d1, copies), dn)
