"""The library's own number of depth slabs follows the call, not the
workspace."""
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu


def _run(sc, cam, dtype="bf16", slabs=None, p=0.5, pair_capacity=0):
    import torch
    from paper_2308_04669_amd import api
    old = api.tune_get("slabs", dtype)
    ws = api.Workspace()
    try:
        if slabs is not None:
            api.tune_set("slabs", dtype, slabs)
        dep, idn = api.infer_depth_id(sc, api.camera_rays(cam), dtype=dtype, p_lo=p, p_hi=p, refine_steps=0, ws=ws,
                                      pair_capacity=pair_capacity)
        torch.cuda.synchronize()
    finally:
        api.tune_set("slabs", dtype, old)
    assert api.check_status(ws) == 0
    st = api.ws_counters(ws)
    return dep, idn, st["culled_pairs"], st["nedf_hits"] + st["fallback"] + st["nedf_misses"]


def test_slabs_do_not_depend_on_the_workspace():
    """The same call evaluates the same pairs in a workspace for every ray
    and instance and in one that just holds the culled pairs."""
    need_gpu()
    import torch
    models, insts, cam, _ = syn.batched_scene(4, 200, 480, 270)
    sc = gpu_scene(models, insts, "bf16", nedf_models=[syn.nedf_model(4, 200 + k, head_scale=16.0)
                                                       for k in range(len(models))])
    d0, i0, culled, e0 = _run(sc, cam, p=0.5)
    d1, i1, _, e1 = _run(sc, cam, p=0.5, pair_capacity=culled)
    log(f"[auto slabs] {culled} culled pairs: {e0} evaluated, {e1} in the tight workspace")
    assert e0 < culled  # several slabs
    assert e0 == e1 and torch.equal(d0, d1) and torch.equal(i0, i1)
