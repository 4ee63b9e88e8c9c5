"""The marcher's samples are decided the same way in every kernel: rays that
graze the bounding sphere of a masked field, where nearly every sample lies
within a rounding of the mask, and rays over the SDF shapes give the same bits
in short lists, in long ones and in every launch shape."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu


def _rays(n, seed, graze):
    """Unit-direction rays from |o| = 4: past the unit sphere's edge at half
    chords of 6e-4 to 6e-3, or at the ball of radius 0.8."""
    g = np.random.default_rng(seed)
    u = g.standard_normal((n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    v = np.cross(u, g.standard_normal((n, 3)))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    b = np.sqrt(1.0 - 10.0 ** g.uniform(2 * np.log10(6e-4), 2 * np.log10(6e-3), n)) if graze else 0.8 * g.random(n)
    d = -u * np.sqrt(1.0 - (b / 4.0) ** 2)[:, None] + v * (b / 4.0)[:, None]
    return (4.0 * u).astype(np.float32), d.astype(np.float32)


@pytest.mark.parametrize("mode", ["softplus", "sdf"])
@pytest.mark.parametrize("samples", [64, 200])
def test_march_same_bits_in_every_kernel(mode, samples):
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    models = [syn.nerf_model(3, 150 + k, sigma_mode=mode, sdf_shape=k) for k in range(4)]
    eye = syn.Instance(0, np.eye(3), np.zeros(3), 1.0)
    n = 240  # fits the kernel of short lists: at most 4 pairs per compute unit
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert n + 1 <= 4 * cus
    copies = -(-6 * cus // n)
    old = api.tune_get("march", "bf16")
    try:
        for k, m in enumerate(models):
            sc = gpu_scene([m], [eye], "bf16")
            o, d = _rays(n, 31 + k, mode == "softplus")

            def run(o, d):
                ws = api.Workspace()
                out = api.march_depth(sc, api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()),
                                      n_samples=samples, dtype="bf16", ws=ws)
                torch.cuda.synchronize()
                return [x.cpu().numpy().view(np.uint32) for x in out], api.ws_counters(ws)["pairs"]

            short, pairs = run(o, d)
            assert 0 < pairs <= 4 * cus - 1
            opac = short[2].view(np.float32)
            log(f"[march bits] {mode}, shape {k}, {samples} samples: {pairs} pairs, "
                f"{int((opac > 0).sum())} with opacity, up to {opac.max():.3g}")
            assert (opac > 0).sum() > n // 4
            for v in api.tune_candidates("march", "bf16"):
                api.tune_set("march", "bf16", v)
                long, pairs = run(np.tile(o, (copies, 1)), np.tile(d, (copies, 1)))
                assert pairs > 4 * cus
                for a, b in zip(short, long):
                    assert np.array_equal(np.tile(a, copies), b), (mode, k, v)
    finally:
        api.tune_set("march", "bf16", old)
