"""Lists of one round of four-wave items and longer ones: the same rays must
give the same bits from either kernel, at ray counts around the kernels' items
of 128 and 256 pairs."""
import numpy as np
import pytest

import synthetic as syn
from tests.gpu_util import need_gpu, gpu_scene, log
from tests.test_gpu_small import _same_in_copies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 127, 257])
@pytest.mark.parametrize("n_blocks", [1, 3])
def test_short_and_long_lists_same_bits_classifier(n, n_blocks):
    need_gpu()
    from paper_2308_04669_amd import api
    models, insts, _ = syn.sdf_scene(3, 6)
    nets = [syn.classifier_model(3, 500 + k, n_blocks=n_blocks, bias_std=0.05) for k in range(len(models))]
    sc = gpu_scene(models, insts, "bf16", nedf_models=nets)
    log(f"case: classifier lists, {n} rays, {n_blocks} blocks")
    copies = -(-70000 // n)  # beyond 256 items of 128 pairs
    dep, idn = _same_in_copies(lambda r: api.infer_depth_id(sc, r, dtype="bf16", refine_steps=0), n, copies)
    log(f"[classifier lists] {n} rays, {copies} copies: {int((idn >= 0).sum())} hits")


@pytest.mark.parametrize("n", [1, 129])
def test_short_and_long_lists_same_bits_fp8(n):
    """FP8 regression networks: calls that fit one round of four-wave items
    and longer ones (eight waves)."""
    need_gpu()
    import torch
    from paper_2308_04669_amd import api
    models, insts, _ = syn.sdf_scene(3, 6)
    nets = [syn.nedf_model(3, 200 + k, head_scale=4.0) for k in range(len(models))]
    o, d = syn.training_rays(3, 42, 1024)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
    objs = []
    for m, net in zip(models, nets):
        scales = api.fp8_calibrate(net.trunk.W, net.trunk.b, t(o), t(d), enc_L=8).reshape(-1)
        objs.append(api.object_from_model(m, "bf16", nedf_model=net, nedf_dtype="fp8", nedf_scales=scales))
    sc = api.make_scene(objs, insts)
    log(f"case: FP8 lists, {n} rays")
    dep, idn = _same_in_copies(lambda r: api.infer_depth_id(sc, r, dtype="bf16", refine_steps=0), n, -(-40000 // n))
    log(f"[fp8 lists] {n} rays: {int((idn >= 0).sum())} hits")
