"""Counters of the depth calls (nedf_ws_counters)."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", ["sphere", "nerf"])
def test_keys_count_the_marched_pairs(field):
    """infer_keys reports the same routing and marched pairs as
    infer_depth_id on the same scene."""
    need_gpu()
    from paper_2308_04669_amd import api
    models, insts, cam = syn.sdf_scene(3, 6, width=48, height=40)
    if field == "sphere":
        models = [syn.Model(kind="sphere", bound=1.0, params=dict(syn.SPHERE_A)) for _ in models]
    nets = [syn.nedf_model(3, 200 + k, head_scale=4.0) for k in range(len(models))]
    sc = api.make_scene([api.object_from_model(m, "bf16", nedf_model=n) for m, n in zip(models, nets)], insts)
    rays = api.camera_rays(cam)
    ws, wk = api.Workspace(), api.Workspace()
    api.infer_depth_id(sc, rays, dtype="bf16", refine_steps=0, ws=ws)
    api.infer_keys(sc, rays, dtype="bf16", ws=wk)
    full, keys = api.ws_counters(ws), api.ws_counters(wk)
    log(f"[counters] {field}: {full}")
    assert full["fallback_marched"] > 0
    assert keys == full
