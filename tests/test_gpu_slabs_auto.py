"""The library's own number of depth slabs follows the pairs that culling
keeps, not the workspace; whatever the number, the results are those of one
slab."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log

pytestmark = pytest.mark.gpu


def _stack(n_inst, width, height, dtype="bf16", cls=False):
    """Instances of three quarters of the image each, behind one another,
    with networks that report a hit wherever they run."""
    models = [syn.nerf_model(4, 100, sigma_mode="sdf", sdf_shape=0)]
    net = syn.classifier_model(4, 500, n_blocks=2, bias_std=0.05) if cls else syn.nedf_model(4, 200, head_scale=16.0)
    g = syn.rng(4, 950)
    insts = []
    for k in range(n_inst):
        z = 6.0 + 24.0 * k / n_inst
        insts.append(syn.Instance(0, syn.shoemake_rotation(g),
                                  np.array([g.uniform(-0.1, 0.1) * z, g.uniform(-0.1, 0.1) * z, -z]), 0.3 * z))
    cam = syn.Camera(eye=(0.0, 0.0, 0.0), at=(0.0, 0.0, -1.0), up=(0.0, 1.0, 0.0), fov_y_deg=40.0, width=width,
                     height=height)
    return gpu_scene(models, insts, dtype, nedf_models=[net]), cam


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


@pytest.mark.parametrize("dtype,width,height,n_inst", [("bf16", 320, 180, 60), ("f32", 160, 90, 60)])
def test_many_objects_along_a_ray_are_pruned(dtype, width, height, n_inst):
    """Where culling keeps most pairs, the automatic number of slabs skips
    hidden ones; few pairs are evaluated in one slab."""
    need_gpu()
    import torch
    sc, cam = _stack(n_inst, width, height, dtype)
    d0, i0, culled, e0 = _run(sc, cam, dtype)
    d1, i1, _, e1 = _run(sc, cam, dtype, slabs=1)
    log(f"[auto slabs] {dtype} {width} x {height}, {n_inst} instances: {e0} of {culled} pairs evaluated")
    assert torch.equal(d0, d1) and torch.equal(i0, i1)
    assert e1 == culled and e0 < 0.7 * culled
    sc, cam = _stack(4, 64, 64, dtype)
    _, _, culled, e = _run(sc, cam, dtype)
    assert e == culled


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


@pytest.mark.parametrize("cls", [False, True])
def test_slabs_of_long_lists_same_bits(cls):
    """More than 8.4 M culled pairs: every wave of the slab filters takes
    several blocks of 1,024 pairs and carries candidates from one to the next."""
    need_gpu()
    import torch
    sc, cam = _stack(32, 1280, 720, cls=cls)
    d1, i1, culled, e1 = _run(sc, cam, slabs=1)
    assert culled > 8.4e6 and e1 == culled
    for v in (2, 4, 32):
        d, i, _, e = _run(sc, cam, slabs=v)
        log(f"[long slabs] {v} slabs: {e} of {culled} pairs evaluated")
        assert e < e1 and torch.equal(d, d1) and torch.equal(i, i1)
