"""Composition in a workspace that holds the pixels of either kind of refined
object (analytic and network), but not both at once."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, log

pytestmark = pytest.mark.gpu


def test_compose_refines_each_kind_within_the_capacity():
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    nerf = syn.nerf_model(3, 150, sigma_mode="sdf", sdf_shape=0)
    net = syn.nedf_model(3, 200, head_scale=4.0)
    objs = [api.ObjectSpec("sphere", 1.0, (50.0, 0.7, 0.01, 0.8, 0.8, 0.8)),
            api.object_from_model(nerf, "bf16", nedf_model=net)]
    insts = [syn.Instance(0, np.eye(3), np.array([-1.1, 0.0, -4.0]), 1.0),
             syn.Instance(1, np.eye(3), np.array([1.1, 0.0, -4.0]), 1.0)]
    sc = api.make_scene(objs, insts)
    cam = syn.Camera(eye=(0.0, 0.0, 0.0), at=(0.0, 0.0, -1.0), up=(0.0, 1.0, 0.0), fov_y_deg=32.0, width=192, height=96)
    rays = api.camera_rays(cam)
    # p_lo = 0, p_hi = 1: the network's pairs are marched, which hits the sphere of its field
    keys = api.infer_keys(sc, rays, dtype="bf16", p_lo=0.0, p_hi=1.0)
    ref, ids = api.compose_keys(sc, rays, [keys], dtype="bf16")
    kinds = [int((ids == k).sum()) for k in range(2)]
    cap = -(-max(kinds) // 1024) * 1024
    ws = api.Workspace()
    dep, idn = api.compose_keys(sc, rays, [keys], dtype="bf16", ws=ws, pair_capacity=cap)
    torch.cuda.synchronize()
    log(f"[compose] {kinds} pixels to refine, capacity {cap}, {int((dep != ref).sum())} depths differ")
    assert min(kinds) > 1024 and sum(kinds) > cap + 1024
    assert api.check_status(ws) == 0
    assert torch.equal(ids, idn) and torch.equal(ref, dep)
    assert api.ws_counters(ws)["pairs"] == kinds[1]  # the networks' pixels
