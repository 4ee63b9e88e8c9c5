"""Which kernel takes a list: short and long lists of the same rays have to
reach both kernels of each stage (shown by the counters) and give the same
bits, and short lists of large calls run on the short lists' kernels too."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log
from tests.test_gpu_small import _rays

pytestmark = pytest.mark.gpu


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _query(sc, o, d, dtype, **kw):
    import torch
    from paper_2308_04669_amd import api
    ws = api.Workspace()
    rays = api.array_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
    dep, idn = api.infer_depth_id(sc, rays, dtype=dtype, ws=ws, **kw)
    torch.cuda.synchronize()
    return dep.cpu().numpy().view(np.uint32), idn.cpu().numpy(), api.ws_counters(ws)


def _query_one_slab(sc, o, d, dtype, **kw):
    """All pairs in one list of the network stage."""
    from paper_2308_04669_amd import api
    old = api.tune_get("slabs", dtype)
    try:
        api.tune_set("slabs", dtype, 1)
        return _query(sc, o, d, dtype, **kw)
    finally:
        api.tune_set("slabs", dtype, old)


def _scene(dtype, cls=False):
    models, insts, _ = syn.sdf_scene(3, 6)
    nets = [syn.classifier_model(3, 500 + k, n_blocks=2, bias_std=0.05) if cls else syn.nedf_model(3, 200 + k)
            for k in range(len(models))]
    return gpu_scene(models, insts, dtype, nedf_models=nets), len(models)


@pytest.mark.parametrize("n", [33, 257])
@pytest.mark.parametrize("stage", ["march", "refine", "net", "net_cls", "net_f32"])
def test_both_kernels_of_a_stage_same_bits(stage, n):
    need_gpu()
    dtype = "f32" if stage == "net_f32" else "bf16"
    sc, n_obj = _scene(dtype, stage == "net_cls")
    # every pair marched (p_lo = 0, p_hi = 1), or none
    kw = dict(p_lo=0.0, p_hi=1.0) if stage in ("march", "refine") else dict(p_lo=0.0, p_hi=0.0)
    kw["refine_steps"] = 3 if stage == "refine" else 0
    kw["n_samples"] = 40
    # the short lists' kernel: pairs of its units, and most units
    unit, units = {"march": (1, 4), "refine": (32, 3), "net": (32, 3), "net_cls": (128, 1), "net_f32": (32, 36)}[stage]
    most = unit * units * _cus()
    o, d = _rays(n, 17 + n)

    def listed(st):
        return {"march": st["fallback_marched"], "refine": st["pairs"]}.get(stage, st["culled_pairs"])

    query = _query_one_slab if stage.startswith("net") else _query
    d1, i1, st1 = query(sc, o, d, dtype, **kw)
    copies = -(-2 * most // max(1, listed(st1)))
    dn, idn, stn = query(sc, np.tile(o, (copies, 1)), np.tile(d, (copies, 1)), dtype, **kw)
    log(f"[list routes] {stage}, {n} rays: {listed(st1)} and {listed(stn)} pairs about the limit {most}")
    assert 0 < listed(st1) <= most - unit * n_obj and listed(stn) > most
    if stage.startswith("net"):
        assert st1["nedf_hits"] > 0 and (stage != "net" or stn["culled_pairs"] == stn["nedf_hits"] + stn["nedf_misses"] + stn["fallback"])
    assert np.array_equal(np.tile(i1, copies), idn) and np.array_equal(np.tile(d1, copies), dn)


def test_short_lists_of_large_calls():
    """A small object in a frame of more than 2^20 rays: its marched and its
    refined pixels take as long as in a frame of slightly fewer."""
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    model, net = syn.nerf_model(3, 150, sigma_mode="sdf", sdf_shape=0), syn.nedf_model(3, 200)
    sc = gpu_scene([model], [syn.Instance(0, np.eye(3), np.array([0.0, 0.0, -60.0]), 0.5)], "bf16", nedf_models=[net])

    def stages(width, height):
        cam = syn.Camera(eye=(0.0, 0.0, 0.0), at=(0.0, 0.0, -1.0), up=(0.0, 1.0, 0.0), fov_y_deg=30.0, width=width,
                         height=height)
        rays, ws, best = api.camera_rays(cam), api.Workspace(), {}
        for _ in range(8):
            api.profile_enable(True)
            api.infer_depth_id(sc, rays, dtype="bf16", p_lo=0.0, p_hi=1.0, ws=ws)
            torch.cuda.synchronize()
            for k, (ms, _) in api.profile_read().items():
                best[k] = min(best.get(k, ms), ms)
        api.profile_enable(False)
        st = api.ws_counters(ws)
        log(f"[large calls] {width} x {height}: {st['fallback_marched']} marched, {st['pairs']} refined, {best}")
        assert 64 < st["pairs"] and st["fallback_marched"] < 4 * _cus()
        return best

    a, b = stages(1000, 1000), stages(1100, 1000)
    for k in ("fallback.mlp", "infer.refine"):
        assert b[k] < 1.7 * a[k], k
