"""The training chain kernels at the edges of their shapes: one layer and the
most, each input width (8 or 16 K-steps), batches of one workgroup and of both
workgroup sizes, one residual block.  Against the FP64 oracle with the
products' operands rounded to bfloat16, in which a rounding that falls the
other way moves single terms only (bounds as for the benchmark's network)."""
import numpy as np
import pytest

import synthetic as syn
from oracle import classifier_loss_and_grads, nedf_loss_and_grads
from tests.gpu_util import need_gpu, log

pytestmark = pytest.mark.gpu


def _run(model, enc_L, in_kind, o, d, D, hit):
    import torch
    from paper_2308_04669_amd import api
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    tr = api.Trainer(model.trunk.W, model.trunk.b, enc_L=enc_L, in_kind=in_kind)
    loss = tr.step(t(o), t(d), t(D), t(hit.astype(np.uint8)), lr=0.0)
    torch.cuda.synchronize()
    gW, gb = tr.export(1)
    return loss.cpu().numpy().astype(np.float64), gW, gb


def _check(loss, gW, gb, ref):
    worst = 0.0
    for i in range(3):
        assert abs(loss[i] - ref[i]) <= 2e-3 * abs(ref[i]) + 1e-7, (i, loss, ref[:3])
    for i, (dw, db) in enumerate(ref[3]):
        assert np.isfinite(gW[i]).all() and np.isfinite(gb[i]).all(), i
        worst = max(worst, np.linalg.norm(gW[i] - dw) / np.linalg.norm(dw),
                    np.linalg.norm(gb[i] - db) / np.linalg.norm(db))
    log(f"worst relative gradient error: {worst:.3e}")
    assert worst <= 3e-2


def _labels(o, d, r=0.5):
    tp = -np.sum(o * d, axis=1)
    b2 = np.sum(o * o, axis=1) - tp ** 2
    hit = b2 < r * r
    D = np.where(hit, tp - np.sqrt(np.maximum(r * r - b2, 0.0)), 0.0).astype(np.float32)
    return D, hit, np.where(hit, tp - D.astype(np.float64), 0.0)


@pytest.mark.parametrize("in_kind,enc_L,depth,B", [
    ("pluecker", 8, 1, 256), ("pluecker", 12, 16, 256), ("pluecker", 0, 2, 512), ("pluecker", 10, 3, 768),
    ("xyz", 12, 3, 256), ("pluecker", 8, 2, 33024), ("pluecker", 12, 2, 33024), ("xyz", 6, 2, 33024)])
def test_line_chain(in_kind, enc_L, depth, B, monkeypatch):
    need_gpu()
    log(f"case: {in_kind} gamma_{enc_L}, {depth} hidden layers, B = {B}")
    model = syn.nedf_model(4, 71, enc_L=enc_L, depth=depth)
    g = syn.rng(4, 72)
    if in_kind == "xyz":
        import oracle.train as T
        monkeypatch.setattr(T, "pluecker", lambda o, d: (o, None))
        w0 = model.trunk.W[0]
        n = 3 * (1 + 2 * enc_L)
        model.trunk.W[0] = (g.standard_normal((w0.shape[0], n)) * np.sqrt(2.0 / n)).astype(np.float32)
    for bb in model.trunk.b:
        bb[:] = (g.standard_normal(bb.shape) * 0.05).astype(np.float32)
    o, d = syn.training_rays(4, 73, B)
    D, hit, mu = _labels(o.astype(np.float64), d.astype(np.float64))
    loss, gW, gb = _run(model, enc_L, in_kind, o, d, D, hit)
    _check(loss, gW, gb, nedf_loss_and_grads(model, o.astype(np.float64), d.astype(np.float64), mu,
                                             hit.astype(np.float64), gemm="bf16"))


@pytest.mark.parametrize("n_blocks,B", [(1, 256), (2, 768), (1, 16640)])  # two waves; four past one round of them
def test_points_chain(n_blocks, B):
    need_gpu()
    log(f"case: classifier, {n_blocks} blocks, B = {B}")
    model = syn.classifier_model(3, 74, n_blocks=n_blocks, bias_std=0.05)
    o, d = syn.training_rays(3, 75, B)
    # labels at the centres of fine bins: the bin does not hang on a rounding
    g = np.random.default_rng(76)
    o64, d64 = o.astype(np.float64), d.astype(np.float64)
    tp = -np.sum(o64 * d64, axis=1)
    hit = g.random(B) < 0.5
    mu_c = (g.integers(0, 64 * 128, B) + 0.5) / (64 * 128) * 2.0 - 1.0
    D = np.where(hit, tp - mu_c, 0.0).astype(np.float32)
    mu = np.where(hit, tp - D.astype(np.float64), 0.0)
    loss, gW, gb = _run(model, 10, "points16", o, d, D, hit)
    _check(loss, gW, gb, classifier_loss_and_grads(model, o64, d64, mu, hit.astype(np.float64), gemm="bf16"))
