"""Depth slabs: a number that is set is the number that runs, and the pruning
between slabs is exact."""
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu


def _run(sc, rays, slabs):
    import torch
    from paper_2308_04669_amd import api
    old = api.tune_get("slabs", "bf16")
    ws = api.Workspace()
    try:
        api.tune_set("slabs", "bf16", slabs)
        dep, idn = api.infer_depth_id(sc, rays, dtype="bf16", refine_steps=0, ws=ws)
        torch.cuda.synchronize()
    finally:
        api.tune_set("slabs", "bf16", old)
    st = api.ws_counters(ws)
    return dep, idn, st, st["nedf_hits"] + st["fallback"] + st["nedf_misses"]


def test_more_slabs_skip_more_pairs():
    """Instances behind one another: the network must run on strictly fewer
    pairs with 2, 4 and 8 slabs each (a number that silently fell back to
    another would not), with the same bits."""
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    models, insts, cam, _ = syn.batched_scene(4, 200, 160, 90)
    nets = [syn.nedf_model(4, 200 + k, head_scale=16.0) for k in range(len(models))]
    sc = gpu_scene(models, insts, "bf16", nedf_models=nets)
    rays = api.camera_rays(cam)
    ref, evald = None, {}
    for v in (1, 2, 4, 8):
        dep, idn, st, evald[v] = _run(sc, rays, v)
        ref = ref or (dep, idn)
        assert torch.equal(dep, ref[0]) and torch.equal(idn, ref[1])
    log(f"[slabs] evaluated pairs {evald} of {st['pairs']}")
    assert evald[1] == st["pairs"] and evald[1] > evald[2] > evald[4] > evald[8]
