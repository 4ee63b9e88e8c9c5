"""The marcher of short (and of all FP32) lists takes samples 64 at a time and
the last 32 or fewer alone: the same samples in another pass give the same
bits, and samples that are not asked for cost nothing."""
import time

import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu

# (samples, t_near): 1/16 apart, so that every form has the object's samples
# (t in [3, 5]) at the same places, exactly, and in the same groups of 32; the
# others see nothing and add exact zeros
FORMS = [[(64, 2), (65, 2), (96, 2), (96, 0), (97, 0), (128, 0), (160, 0)], [(32, 3), (33, 3), (64, 1), (64, 3), (95, 1)]]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("forms", FORMS)
def test_march_same_bits_in_every_pass(dtype, forms):
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    sc = gpu_scene([syn.nerf_model(3, 151)], [syn.Instance(0, np.eye(3), np.zeros(3), 1.0)], dtype)
    g = np.random.default_rng(6)
    n = 200
    o = np.concatenate([g.uniform(-0.7, 0.7, (n, 2)), np.full((n, 1), 4.0)], axis=1).astype(np.float32)
    d = np.tile(np.float32([0.0, 0.0, -1.0]), (n, 1))
    rays = api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
    ref = None
    for samples, t_near in forms:
        out = api.march_depth(sc, rays, n_samples=samples, clip_to_bound=False, t_near=float(t_near),
                              t_far=t_near + samples / 16.0, hit_threshold=1e-3, dtype=dtype)
        torch.cuda.synchronize()
        out = [x.cpu().numpy().view(np.uint32) for x in out]
        ref = ref or out
        opac = out[2].view(np.float32)
        log(f"[march passes] {dtype}, {samples} samples from {t_near}: opacity {opac.min():.3g} .. {opac.max():.3g}")
        assert (opac > 1e-3).all()
        for a, b in zip(ref, out):
            assert np.array_equal(a, b), (samples, t_near)


@pytest.mark.parametrize("samples", [1, 20, 32])
def test_long_f32_lists_of_few_samples_same_bits(samples):
    """Long lists of at most 32 samples take another kernel than short ones."""
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    models, insts, _, _ = syn.config2_scene(n_objects=3)
    sc = gpu_scene(models, insts, "f32")
    g = np.random.default_rng(8)
    n = 250
    o = np.concatenate([g.uniform(-1.0, 1.0, (n, 2)), np.full((n, 1), 13.0)], axis=1).astype(np.float32)
    t = np.concatenate([g.uniform(-3.0, 3.0, (n, 2)), np.zeros((n, 1))], axis=1)
    d = ((t - o) / np.linalg.norm(t - o, axis=1, keepdims=True)).astype(np.float32)
    limit = 36 * torch.cuda.get_device_properties(0).multi_processor_count

    def run(o, d):
        ws = api.Workspace()
        rays = api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
        out = api.march_depth(sc, rays, n_samples=samples, dtype="f32", ws=ws)
        torch.cuda.synchronize()
        return [x.cpu().numpy().view(np.uint32) for x in out], api.ws_counters(ws)["pairs"]

    one, p1 = run(o, d)
    copies = -(-2 * limit // p1)
    many, pn = run(np.tile(o, (copies, 1)), np.tile(d, (copies, 1)))
    log(f"[march lists] f32, {samples} samples: {p1} and {pn} pairs about the limit {limit}, "
        f"opacity up to {one[2].view(np.float32).max():.3f}")
    assert 0 < p1 <= limit - len(models) and pn > limit
    for a, b in zip(one, many):
        assert np.array_equal(np.tile(a, copies), b)


def test_march_f32_time_follows_the_samples():
    """32 samples cost about half of 64, 96 about three quarters of 128."""
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    models, insts, cam, _ = syn.config2_scene(n_objects=8, width=128, height=128)
    sc = gpu_scene(models, insts, "f32")
    rays, ws = api.camera_rays(cam), api.Workspace()

    def ms(samples):
        best = float("inf")
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            api.march_depth(sc, rays, n_samples=samples, dtype="f32", ws=ws)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return 1e3 * best

    t = {n: ms(n) for n in (32, 64, 96, 128)}
    log(f"[march tail] ms by samples: {t}")
    assert t[32] < 0.75 * t[64] and t[96] < 0.87 * t[128]
