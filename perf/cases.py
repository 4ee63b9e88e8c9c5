"""Performance cases: what programs built on this framework have it do, through
``paper_2308_04669_amd.api``, from the smallest calls (launch latency) to full
frames and training batches.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call, ``run``
is one pass, ``work`` the bytes and operations it cannot do without, and
``exact`` the same outputs in float64 (plain torch, none of the framework's
code) where that is feasible and the result is not decided by a threshold
on a 16-bit value.

The scenes are objects whose density is an SDF-biased NeRF (random trunk,
the sphere of radius 0.6 as its signed distance) and whose intersection
network knows that sphere: part of its units is built to compute
mu = sqrt(r^2 - |m|^2) and a hit logit, the others are a dense random
network of ordinary size whose outputs perturb the result a little.  Routing is
then that of trained networks (confident hits and misses, a narrow uncertain
band for the marcher, more when quantised), which random networks do not
give, and nothing has to be trained to prepare a case.
"""
import math
from types import SimpleNamespace as NS

import numpy as np
import torch

from paper_2308_04669_amd import api

R0 = 0.6          # radius of the objects' surface, in bounding radii
KAPPA = 600.0     # slope of the hit logit in r^2 - |m|^2
SIGMA_MAX, SDF_WIDTH = 50.0, 0.01
EXACT_FLOPS = 7e13  # float64 references beyond this many operations are left out
MAC_DENSITY = 63 * 256 + 7 * 256 * 256 + 256
MAC_COLOUR = 283 * 128 + 128 * 3
MAC_NEDF = 102 * 256 + 7 * 256 * 256 + 2 * 256
MAC_CLS = 1008 * 256 + 32 * 256 * 256 + 193 * 256


def listed():
    return [
        # the smallest marcher call: one object with a 3 x 64 density network, a thumbnail of rays
        dict(name="march_f32_32px", kind="march", net="small", dtype="f32", width=32, height=32, n_inst=1, samples=64),
        # reference rendering of 16 NeRFs without intersection networks, every sample evaluated
        dict(name="march_bf16_800px_16obj", kind="march", net="nerf", dtype="bf16", width=800, height=800, n_inst=16,
             samples=192),
        # a picking or preview query on a small scene: launch latency
        dict(name="infer_bf16_64px_8inst", kind="infer", form="line", dtype="bf16", net_dtype="bf16", width=64,
             height=64, n_inst=8),
        # depth and ID of the batched scene at full size
        dict(name="infer_bf16_1080p_1000inst", kind="infer", form="line", dtype="bf16", net_dtype="bf16", width=1920,
             height=1080, n_inst=1000),
        # full-precision queries along arbitrary rays (visibility, collision), a ragged count
        dict(name="infer_f32_20011rays_24inst", kind="infer", form="line", dtype="f32", net_dtype="f32", rays=20011,
             n_inst=24),
        # quantised intersection networks on a 2160p frame
        dict(name="infer_fp8_2160p_64inst", kind="infer", form="line", dtype="bf16", net_dtype="fp8", width=3840,
             height=2160, n_inst=64),
        # the classifier form of the intersection network on the 900 x 600 scenes
        dict(name="infer_cls_900x600_20inst", kind="infer", form="points", dtype="bf16", net_dtype="bf16", width=900,
             height=600, n_inst=20),
        # deferred shading of a full frame, 8 samples per pixel
        dict(name="shade_bf16_1080p_k8", kind="shade", dtype="bf16", width=1920, height=1080, n_inst=200, K=8),
        # one whole frame: transforms, depth and ID, single-sample shading, shadows of two lights
        dict(name="frame_bf16_900x600_100inst", kind="frame", dtype="bf16", width=900, height=600, n_inst=100, K=1),
        # a frame while one object is dragged: the others' depth keys are kept
        dict(name="reuse_bf16_1080p_200inst", kind="reuse", dtype="bf16", width=1920, height=1080, n_inst=200),
        # one training step of the regression form at the usual batch
        dict(name="train_line_65536", kind="train", form="line", batch=65536),
        # one training step of the classifier form, a quarter batch
        dict(name="train_points_16384", kind="train", form="points", batch=16384),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["march", "infer", "infer", "infer", "shade", "frame", "reuse", "train", "train"])
    if kind == "march":
        small = rng.random() < 0.5
        w, h = _spread(rng, 24, 400), _spread(rng, 24, 400)
        return dict(kind=kind, net="small" if small else "nerf", dtype=rng.choice(["f32", "bf16"] if small else ["bf16"]),
                    width=w, height=h, n_inst=1 if small else rng.randint(2, 16), samples=rng.randint(48, 192))
    if kind == "infer":
        form = rng.choice(["line", "line", "line", "points"])
        dtype = rng.choice(["bf16", "bf16", "f32"]) if form == "line" else "bf16"
        net = rng.choice(["bf16", "bf16", "fp8", "fp8mx"]) if form == "line" and dtype == "bf16" else dtype
        case = dict(kind=kind, form=form, dtype=dtype, net_dtype=net)
        if dtype == "f32" or rng.random() < 0.25:
            case.update(rays=_spread(rng, 500, 60000), n_inst=_spread(rng, 2, 64))
        else:
            w = _spread(rng, 48, 1920 if form == "line" else 900)
            case.update(width=w, height=max(33, int(w * rng.uniform(0.5, 1.0))), n_inst=_spread(rng, 4, 300))
        return case
    if kind == "train":
        form = rng.choice(["line", "line", "points"])
        return dict(kind=kind, form=form, batch=256 * (_spread(rng, 4, 256) if form == "line" else _spread(rng, 4, 64)))
    w = _spread(rng, 64, 1920)
    case = dict(kind=kind, dtype="bf16", width=w, height=max(33, int(w * rng.uniform(0.5, 1.0))), n_inst=_spread(rng, 4, 200))
    if kind == "shade":
        case.update(K=rng.choice([1, 2, 4, 8]))
        if rng.random() < 0.25:
            case.update(dtype="f32", width=min(w, 320), height=min(case["height"], 200))
    if kind == "frame":
        case.update(K=rng.choice([1, 8]), width=min(w, 900), height=min(case["height"], 600))
    return case


# ---- objects ---------------------------------------------------------------------
def _normal(g, n_out, n_in, gain):
    return (g.standard_normal((n_out, n_in), dtype=np.float32) * np.float32(math.sqrt(gain / n_in)))


def _mlp(g, dims, gain):
    W = [_normal(g, dims[i + 1], dims[i], gain if i + 2 < len(dims) else 1.0) for i in range(len(dims) - 1)]
    return NS(W=W, b=[np.zeros(w.shape[0], np.float32) for w in W])


def _nerf(g, mode):
    """NeRF-shaped object: gamma_10(x) -> 8 x 256 -> density, colour branch with gamma_4(d)."""
    params = dict(enc_L=10, dir_L=4, sigma_mode=mode, masked=True)
    if mode == "sdf":
        params.update(sdf_shape=0, sigma_max=SIGMA_MAX, width=SDF_WIDTH)
    return NS(kind="nerf", bound=1.0, params=params, trunk=_mlp(g, [63] + [256] * 8 + [1], 1.0),
              rgb=_mlp(g, [283, 128, 3], 1.0))


def _small_mlp(g):
    return NS(kind="mlp", bound=1.0, params=dict(enc_L=6, sigma_mode="softplus", masked=False),
              trunk=_mlp(g, [39, 64, 64, 64, 1], 1.0), rgb=None)


Q_KNOTS = np.array([0.0, 0.09, 0.17, 0.23, 0.27, 0.30, 0.32, 0.335, 0.346, 0.353, 0.358, 0.36])  # in |m|^2, r^2 = 0.36
M_KNOTS = np.arange(8) / 8.0


def _square_units(W, inputs):
    """Rows of W (input weights) for 48 units relu(+-x_i - k / 8) of three inputs, their biases, and the weights with
    which the units add up to x_0^2 + x_1^2 + x_2^2 (piecewise linear)."""
    bias, coef, u = np.zeros(W.shape[0], np.float32), np.zeros(48, np.float32), 0
    for cols in inputs:
        for sign in (1.0, -1.0):
            for k, t in enumerate(M_KNOTS):
                W[u, :] = 0.0
                W[u, cols] = sign / len(cols)
                bias[u] = -t
                coef[u] = 0.125 if k == 0 else 0.25
                u += 1
    return bias, coef


def _mu_coef():
    """Weights on relu(q - knot) that give sqrt(r^2 - q) - r at the knots and stay there beyond the last."""
    mu = np.sqrt(R0 * R0 - Q_KNOTS)
    slope = np.diff(mu) / np.diff(Q_KNOTS)
    return np.diff(np.concatenate([[0.0], slope, [0.0]])).astype(np.float32)


def _line_net(g):
    """Intersection network on (d, o x d): gamma_8 -> 8 x 256 -> (mu, hit logit)."""
    t = _mlp(g, [102] + [256] * 8 + [2], 2.0)
    nq = len(Q_KNOTS)
    bias, coef = _square_units(t.W[0], [[3], [4], [5]])
    t.b[0] = bias
    for l in range(1, 8):
        built = 48 if l == 1 else nq
        t.W[l][nq:, :built] = 0.0
        t.W[l][:nq, :] = 0.0
        if l == 1:
            t.W[l][:nq, :48] = coef
            t.b[l][:nq] = -Q_KNOTS
        else:
            t.W[l][:nq, :nq] = np.eye(nq)
    # the random part's share of mu stays small; of the logit it is a few units, which spreads the steps of quantised q
    t.W[8] *= np.float32([[0.01], [10.0]])
    t.W[8][:, :nq] = 0.0
    t.W[8][0, :nq] = _mu_coef()
    t.W[8][1, 0] = -KAPPA
    t.b[8][:] = (R0, KAPPA * R0 * R0)
    return NS(kind="nedf", bound=1.0, params=dict(enc_L=8), trunk=t)


def _points_net(g, n_blocks=16):
    """Intersection network in the classifier form: 16 points -> 256, residual blocks, 1 + 64 + 128 logits.
    The tangency point is the mean of points 7 and 8 on the line."""
    W = [_normal(g, 256, 1008, 2.0)]
    for _ in range(n_blocks):
        W += [_normal(g, 256, 256, 2.0), _normal(g, 256, 256, 2.0 / 16)]
    W.append(_normal(g, 193, 256, 1.0))
    b = [np.zeros(w.shape[0], np.float32) for w in W]
    nq = len(Q_KNOTS)
    keep = 48 + nq  # stream units 0..47 hold the squares, 48..keep-1 the knots of q, the rest is the random network
    bias, coef = _square_units(W[0], [[63 * 7 + i, 63 * 8 + i] for i in range(3)])
    W[0][48:keep, :] = 0.0
    b[0] = bias
    for k in range(n_blocks):
        for w in (W[1 + 2 * k], W[2 + 2 * k]):
            w[:keep, :] = 0.0
            w[:, :keep] = 0.0
        if k == 0:
            W[1][48:keep, :48] = coef
            b[1][48:keep] = -Q_KNOTS
            W[2][48:keep, 48:keep] = np.eye(nq)
    tail, tb = W[-1], b[-1]
    tail[1:65] *= 0.002
    tail[:65, :keep] = 0.0
    tail[0, :] *= 0.01
    tail[0, 48] = -KAPPA
    tb[0] = KAPPA * R0 * R0
    # coarse bin c wins when mu is nearest its centre: logits 2 mu centre - centre^2, linear in mu
    centre = (np.arange(64) + 0.5) / 32.0 - 1.0
    tail[1:65, 48:keep] = 8.0 * 2.0 * centre[:, None] * _mu_coef()[None, :]
    tb[1:65] = 8.0 * (2.0 * centre * R0 - centre ** 2)
    return NS(kind="nedf16", bound=1.0, params=dict(enc_L=10, n_blocks=n_blocks), trunk=NS(W=W, b=b))


# ---- scenes ----------------------------------------------------------------------
def _rotation(g):
    u1, u2, u3 = g.random(3)
    a, b = math.sqrt(1 - u1), math.sqrt(u1)
    x, y, z, w = (a * math.sin(2 * math.pi * u2), a * math.cos(2 * math.pi * u2), b * math.sin(2 * math.pi * u3),
                  b * math.cos(2 * math.pi * u3))
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                     [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                     [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])


LIGHTS = ((20.0, 30.0, 10.0), (-25.0, 20.0, 5.0))


def _scene(case, seed):
    """Models, instances, camera (or rays) of a case: plain host data."""
    g = np.random.Generator(np.random.PCG64([seed, case["n_inst"]]))
    n_inst = case["n_inst"]
    S = NS(g=g, models=[], nets=None, insts=[], cam=None, rays=None)
    if case["kind"] == "march":
        small = case["net"] == "small"
        S.models = [_small_mlp(g) if small else _nerf(g, "softplus") for _ in range(n_inst)]
        for k in range(n_inst):
            S.insts.append(NS(model=k, R=np.eye(3) if small else _rotation(g),
                              T=np.zeros(3) if small else g.uniform(-3, 3, 3), s=1.0 if small else g.uniform(0.5, 1.5)))
        S.cam = NS(eye=(0.0, 0.0, 4.0 if small else 13.0), at=(0.0, 0.0, 0.0), up=(0.0, 1.0, 0.0), fov_y_deg=40.0,
                   width=case["width"], height=case["height"])
        return S
    # instances of up to four models with uneven screen coverage, in front of a camera looking along -z
    S.models = [_nerf(g, "sdf") for _ in range(min(4, n_inst))]
    if case["kind"] != "shade":
        S.nets = [(_points_net if case.get("form") == "points" else _line_net)(g) for _ in S.models]
    W, H = case.get("width", 640), case.get("height", 480)
    f = 0.5 * H / math.tan(math.radians(20.0))
    S.cover = 0.0
    for k in range(n_inst):
        c, z, u, v = g.uniform(0.01, 0.20), g.uniform(6.0, 30.0), g.uniform(0, W), g.uniform(0, H)
        S.cover += c
        S.insts.append(NS(model=k % len(S.models), R=_rotation(g), s=z * math.sqrt(c * W * H / math.pi) / f,
                          T=np.array([(u - 0.5 * W) / f * z, (0.5 * H - v) / f * z, -z])))
    if "rays" in case:  # towards the instances, from all around
        n = case["rays"]
        at = np.array([i.T for i in S.insts])[g.integers(0, n_inst, n)] + 2.0 * g.standard_normal((n, 3))
        o = np.array([0.0, 0.0, -18.0]) + 40.0 * _unit(g.standard_normal((n, 3)))
        S.rays = o.astype(np.float32), _unit(at - o).astype(np.float32)
    else:
        S.cam = NS(eye=(0.0, 0.0, 0.0), at=(0.0, 0.0, -1.0), up=(0.0, 1.0, 0.0), fov_y_deg=40.0, width=W, height=H)
    return S


def _unit(v):
    return v / np.linalg.norm(v, axis=-1, keepdims=True)


def _local_rays(g, n):
    """Training rays: from the sphere of radius 4 towards the ball of radius 1.2."""
    o = 4.0 * _unit(g.standard_normal((n, 3)))
    p = 1.2 * _unit(g.standard_normal((n, 3))) * g.random((n, 1)) ** (1.0 / 3.0)
    return o.astype(np.float32), _unit(p - o).astype(np.float32)


def _extent(S):
    c = np.mean([i.T for i in S.insts], axis=0)
    return 2.0 * max(float(np.linalg.norm(i.T - c)) + i.s for i in S.insts)


# ---- prepare ---------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "train":
        return _prepare_train(case, seed)
    S = _scene(case, seed)
    st = NS(case=case, out=None)
    nd = case.get("net_dtype", case["dtype"])
    objs = []
    for i, m in enumerate(S.models):
        net, scales = (S.nets[i] if S.nets else None), None
        if nd == "fp8":
            o, d = _local_rays(S.g, 4096)
            scales = api.fp8_calibrate(net.trunk.W, net.trunk.b, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
        objs.append(api.object_from_model(m, case["dtype"], nedf_model=net, nedf_dtype=nd, nedf_scales=scales))
    st.scene = api.make_scene(objs, S.insts)
    if S.cam is not None:
        st.rays = api.camera_rays(S.cam)
    else:
        st.rays = api.array_rays(torch.from_numpy(S.rays[0]).cuda(), torch.from_numpy(S.rays[1]).cuda())
    n = api.n_rays(st.rays)
    st.ws, st.lights, st.eps = api.Workspace(), LIGHTS, 0.01 * _extent(S)
    # large scenes: pair lists for the pairs that the instances' coverage gives, not for rays x instances
    st.cap = int(1.1 * S.cover * n) + (1 << 20) if n * case["n_inst"] > 1 << 29 else 0
    st.depth = torch.empty(n, dtype=torch.float32, device="cuda")
    st.ident = torch.empty(n, dtype=torch.int32, device="cuda")
    st.rgb = torch.empty((n, 3), dtype=torch.float32, device="cuda")
    st.fac = torch.empty(n, dtype=torch.float32, device="cuda")
    if case["kind"] == "march":
        st.opacity = torch.empty(n, dtype=torch.float32, device="cuda")
    if case["kind"] == "shade":  # the depth and ID buffers of the stage before: nearest surface sphere
        o, d = _rays64(S)
        best = torch.full((n,), math.inf, dtype=torch.float64, device="cuda")
        ident = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        for k, i in enumerate(S.insts):
            c = torch.tensor(i.T, device="cuda") - o
            tp = (c * d).sum(1)
            h2 = (R0 * i.s) ** 2 - ((c * c).sum(1) - tp * tp)
            t = torch.where(h2 > 0, tp - h2.clamp_min(0).sqrt(), math.inf)
            near = t < best
            best, ident = torch.where(near, t, best), torch.where(near, k, ident)
        st.depth, st.ident = best.float(), ident
    if case["kind"] == "reuse":  # instance 0 moves a little; the others' keys are those of the last frames
        G = st.scene.inst_G.clone()
        G[0, 9] += 0.02 * _extent(S)
        st.moved = api.SceneGPU(st.scene.objects, st.scene.inst_object, G, api.compose_transforms(G))
        rest, gid = api.subset_scene(st.moved, range(1, case["n_inst"]))
        st.keys = api.infer_keys(rest, st.rays, gid, dtype=case["dtype"], ws=api.Workspace(), pair_capacity=st.cap)
        st.sub, st.gid = api.subset_scene(st.moved, [0])
        st.ws2, st.keys2 = api.Workspace(), torch.empty_like(st.keys)
    return st


def _prepare_train(case, seed):
    g = np.random.Generator(np.random.PCG64([seed, case["batch"]]))
    points, B = case["form"] == "points", case["batch"]
    if points:
        W = [_normal(g, 256, 1008, 2.0)]
        for _ in range(16):
            W += [_normal(g, 256, 256, 2.0), _normal(g, 256, 256, 2.0 / 16)]
        W.append(_normal(g, 193, 256, 1.0))
    else:
        W = _mlp(g, [102] + [256] * 8 + [2], 2.0).W
    # biases that have left zero, as after the first epochs
    b = [np.float32(0.05) * g.standard_normal(w.shape[0], dtype=np.float32) for w in W]
    o, d = _local_rays(g, B)
    # labels of the sphere, as a marcher gives them for every ray
    tp = -np.sum(o.astype(np.float64) * d, axis=1)
    h2 = R0 * R0 - (np.sum(o.astype(np.float64) ** 2, axis=1) - tp * tp)
    hit = h2 > 0
    depth = np.where(hit, tp - np.sqrt(np.maximum(h2, 0)), 0.0)
    st = NS(case=case, W=W, b=b, o=torch.from_numpy(o).cuda(), d=torch.from_numpy(d).cuda(),
            depth=torch.from_numpy(depth.astype(np.float32)).cuda(), hit=torch.from_numpy(hit.astype(np.uint8)).cuda())
    st.trainer = api.Trainer(W, b, enc_L=10 if points else 8, in_kind="points16" if points else "pluecker")
    st.views = _state_views(st.trainer)
    return st


def _state_views(tr):
    """Float32 views of a trainer's state buffer: weights, biases and the last step's gradients of the first layer, the
    equal layers after it (stacked) and the last layer.  Layer: W, its two Adam moments and gradient, b, its moments and
    gradient, two bfloat16 copies of W with K padded to 128, each at a multiple of 256 bytes from offset 256 on."""
    dims = list(tr.dims)
    rows = [256 if len(dims) > 9 else n for n, _ in dims]  # the classifier's last layer is kept with 256 rows
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    f, off, at = tr.state.view(torch.float32), 256, []
    for (_, k), n in zip(dims, rows):
        w, b, h = up(n * k * 4), up(n * 4), up(n * ((k + 127) // 128 * 128) * 2)
        at.append((off, off + 3 * w, off + 4 * w, off + 4 * w + 3 * b))
        off += 4 * w + 4 * b + 2 * h
    out = {}
    for j, name in enumerate(("W", "gW", "b", "gb")):
        def view(i, j=j):
            n, k = dims[i]
            return f[at[i][j] // 4:][:n * k].view(n, k) if j < 2 else f[at[i][j] // 4:][:n]
        mid = view(1)
        out[name] = [view(0), mid.as_strided((len(dims) - 2, *mid.shape), ((at[2][j] - at[1][j]) // 4, *mid.stride())),
                     view(len(dims) - 1)]
    return out


# ---- run -------------------------------------------------------------------------
def run(st):
    c, kind = st.case, st.case["kind"]
    if kind == "train":
        loss = st.trainer.step(st.o, st.d, st.depth, st.hit)
        return dict(loss=loss, **st.views)
    dt = c["dtype"]
    if kind == "march":
        small = c["net"] == "small"
        api.march_depth(st.scene, st.rays, n_samples=c["samples"], clip_to_bound=not small, t_near=2.0 if small else 0.0,
                        t_far=6.0 if small else 0.0, dtype=dt, ws=st.ws, out=(st.depth, st.ident, st.opacity))
        return dict(depth=st.depth, ident=st.ident, opacity=st.opacity)
    if kind == "infer":
        api.infer_depth_id(st.scene, st.rays, dtype=dt, ws=st.ws, pair_capacity=st.cap, out=(st.depth, st.ident))
        return dict(depth=st.depth, ident=st.ident)
    if kind == "shade":
        api.shade_deferred(st.scene, st.rays, st.depth, st.ident, K=c["K"], dtype=dt, ws=st.ws, out=st.rgb)
        return dict(rgb=st.rgb)
    if kind == "reuse":
        api.infer_keys(st.sub, st.rays, st.gid, dtype=dt, ws=st.ws2, out=st.keys2)
        api.compose_keys(st.moved, st.rays, [st.keys, st.keys2], dtype=dt, ws=st.ws, out=(st.depth, st.ident))
        return dict(depth=st.depth, ident=st.ident)
    st.scene.inst_w2l = api.compose_transforms(st.scene.inst_G)
    api.infer_depth_id(st.scene, st.rays, dtype=dt, ws=st.ws, pair_capacity=st.cap, out=(st.depth, st.ident))
    api.shade_deferred(st.scene, st.rays, st.depth, st.ident, K=c["K"], dtype=dt, ws=st.ws, out=st.rgb)
    api.shadow(st.scene, st.rays, st.depth, st.ident, st.lights, st.eps, dtype=dt, ws=st.ws, rgb_inout=st.rgb, out=st.fac)
    return dict(depth=st.depth, ident=st.ident, shadow=st.fac, rgb=st.rgb)


# ---- work ------------------------------------------------------------------------
def work(case):
    """Every pixel is taken to be covered (the scenes cover nearly all of the image): one intersection-network pair per
    ray and light, the secant's four field evaluations, K shading samples.  Pruned pairs, the marcher fallback and
    intermediate buffers are not counted."""
    kind = case["kind"]
    if kind == "train":
        B, points = case["batch"], case["form"] == "points"
        mac = MAC_CLS if points else MAC_NEDF
        params = 2413249 if points else 102 * 256 + 7 * 65536 + 512 + 8 * 256 + 2
        first = (1008 if points else 102) * 256  # the first layer needs no input gradient
        return dict(bytes=float(B * 29 + params * 4 * 7), flops=2.0 * B * (3 * mac - first))
    n = case["rays"] if "rays" in case else case["width"] * case["height"]
    rays = n * 24 if "rays" in case else 0
    blob = {"f32": 4, "bf16": 2}.get(case["dtype"], 1) * 5e5 * min(4, case["n_inst"])
    if kind == "march":
        small = case["net"] == "small"
        mac = 39 * 64 + 2 * 64 * 64 + 64 if small else MAC_DENSITY
        # 16 objects in a cube of 6: a mean chord of two thirds of the diameter over about 7 % of the image each
        pairs = n if small else n * case["n_inst"] * 0.035
        return dict(bytes=float(n * 12 + blob), flops=2.0 * pairs * case["samples"] * mac)
    mac = 0.0
    if kind in ("infer", "frame"):
        mac += MAC_CLS if case.get("form") == "points" else MAC_NEDF
    if kind in ("infer", "frame", "reuse"):
        mac += 4 * MAC_DENSITY
    if kind in ("shade", "frame"):
        mac += case["K"] * (MAC_DENSITY + MAC_COLOUR)
    if kind == "frame":
        mac += 2 * MAC_NEDF
    per = dict(infer=8, shade=8 + 12, reuse=8 + 8, frame=8 + 4 + 12)[kind]
    return dict(bytes=float(n * per + rays + blob + case["n_inst"] * 64), flops=2.0 * n * mac)


# ---- float64 references ----------------------------------------------------------
def _t(x):
    return torch.as_tensor(np.asarray(x, np.float64), device="cuda")


def _rays64(S):
    if S.rays is not None:
        return _t(S.rays[0]), _t(S.rays[1])
    c = S.cam
    eye, up = _t(c.eye), _t(c.up)
    f = _t(c.at) - eye
    f = f / f.norm()
    r = torch.linalg.cross(f, up)
    r = r / r.norm()
    u = torch.linalg.cross(r, f)
    th = math.tan(math.radians(c.fov_y_deg) / 2)
    x = (2 * (torch.arange(c.width, device="cuda", dtype=torch.float64) + 0.5) / c.width - 1) * th * c.width / c.height
    y = (1 - 2 * (torch.arange(c.height, device="cuda", dtype=torch.float64) + 0.5) / c.height) * th
    d = (f + x[None, :, None] * r + y[:, None, None] * u).reshape(-1, 3)
    return eye.expand_as(d), d / d.norm(dim=1, keepdim=True)


def _enc(p, L):
    out = [p]
    for l in range(L):
        a = (2.0 ** l) * math.pi * p
        out += [torch.sin(a), torch.cos(a)]
    return torch.cat(out, dim=1)


class _Net:
    def __init__(self, t):
        self.W, self.b = [_t(w) for w in t.W], [_t(x) for x in t.b]

    def trunk(self, h):
        for W, b in zip(self.W[:-1], self.b[:-1]):
            h = torch.relu(torch.addmm(b, h, W.T))
        return h, torch.addmm(self.b[-1], h, self.W[-1].T)


class _Field:
    """Density of a model at local points, in blocks."""

    def __init__(self, m):
        self.m, self.net = m, _Net(m.trunk)
        self.rgb = _Net(m.rgb) if m.rgb is not None else None

    def surface(self, x):
        return self.net.trunk(_enc(x, self.m.params["enc_L"]))[1][:, 0] - (x.norm(dim=1) - R0) / SDF_WIDTH

    def both(self, x, d=None):
        h, u = self.net.trunk(_enc(x, self.m.params["enc_L"]))
        u, p = u[:, 0], self.m.params
        if p["sigma_mode"] == "sdf":
            s = SIGMA_MAX * torch.sigmoid(u - (x.norm(dim=1) - R0) / SDF_WIDTH)
        else:
            s = torch.nn.functional.softplus(u)
            s = torch.where(x.norm(dim=1) <= 1.0, s, 0.0) if p["masked"] else s
        c = None if d is None else torch.sigmoid(self.rgb.trunk(torch.cat([h, _enc(d, p["dir_L"])], 1))[1])
        return s, c


def _local(i, o, d):
    Rm = _t(i.R)
    return (o - _t(i.T)) @ Rm / i.s, d @ Rm


def _chord(ol, dl):
    tp = -(ol * dl).sum(1)
    h2 = 1.0 - ((ol * ol).sum(1) - tp * tp)
    h = h2.clamp_min(0).sqrt()
    a = (tp - h).clamp_min(0)
    return tp, a, tp + h, (h2 > 0) & (tp + h > a)


def _march(field, ol, dl, a, b, N):
    """Opacity and local depth of segments [a, b]."""
    A, D = torch.zeros_like(a), torch.zeros_like(a)
    step = max(1, (1 << 20) // N)
    for q in range(0, a.numel(), step):
        s = slice(q, q + step)
        dt = ((b[s] - a[s]) / N)[:, None]
        t = a[s, None] + (torch.arange(N, device="cuda", dtype=torch.float64) + 0.5) * dt
        x = ol[s, None] + t[..., None] * dl[s, None]
        v = field.both(x.reshape(-1, 3))[0].view(t.shape) * dt
        w = torch.exp(-(v.cumsum(1) - v)) * -torch.expm1(-v)
        A[s] = w.sum(1)
        D[s] = (w * t).sum(1) / A[s]
    return A, D


def exact(case, seed):
    if work(case)["flops"] > EXACT_FLOPS:
        return None
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] not in ("march", "shade") and not (case["kind"] == "infer" and case["dtype"] == "f32"):
        return None  # which pairs hit is decided by thresholds on 16-bit networks
    S = _scene(case, seed)
    o, d = _rays64(S)
    n = o.shape[0]
    inf = torch.full((n,), math.inf, dtype=torch.float64, device="cuda")
    fields = [_Field(m) for m in S.models]
    if case["kind"] == "march":
        small, depth, opac = case["net"] == "small", inf.clone(), torch.zeros_like(inf)
        for i in S.insts:
            ol, dl = _local(i, o, d)
            if small:
                a, b, at = torch.full_like(inf, 2.0), torch.full_like(inf, 6.0), torch.arange(n, device="cuda")
            else:
                _, a, b, ok = _chord(ol, dl)
                at = ok.nonzero()[:, 0]
            A, D = _march(fields[i.model], ol[at], dl[at], a[at], b[at], case["samples"])
            opac[at] = torch.maximum(opac[at], A)
            depth[at] = torch.minimum(depth[at], torch.where(A >= 0.5, i.s * D, math.inf))
        return dict(depth=depth if case["dtype"] == "f32" else None, ident=None, opacity=opac)
    if case["kind"] == "shade":
        st = prepare(dict(case), seed)  # its depth and ID buffers, made here in float64
        rgb, K, h = torch.zeros((n, 3), dtype=torch.float64, device="cuda"), case["K"], 0.05
        for k, i in enumerate(S.insts):
            for at in (st.ident == k).nonzero()[:, 0].split((1 << 20) // K):
                ol, dl = _local(i, o[at], d[at])
                D, dt = st.depth[at].double(), 2 * h / K
                t = (D[:, None] - h + (torch.arange(K, device="cuda", dtype=torch.float64) + 0.5) * dt) / i.s
                x = ol[:, None] + t[..., None] * dl[:, None]
                s, c = fields[i.model].both(x.reshape(-1, 3), dl[:, None].expand_as(x).reshape(-1, 3))
                v, c = s.view(-1, K) * (dt / i.s), c.view(-1, K, 3)
                w = torch.exp(-(v.cumsum(1) - v)) * -torch.expm1(-v)
                sw = w.sum(1, keepdim=True)
                rgb[at] = torch.where(sw < 1e-6, c[:, (K - 1) // 2], (w[..., None] * c).sum(1) / sw)
        return dict(rgb=rgb)
    best, who = inf.clone(), torch.full((n,), -1, device="cuda")
    nets = [_Net(m.trunk) for m in S.nets]
    for k, i in enumerate(S.insts):
        ol, dl = _local(i, o, d)
        tp, a, b, ok = _chord(ol, dl)
        at = ok.nonzero()[:, 0]
        ol, dl, tp, a, b = ol[at], dl[at], tp[at], a[at], b[at]
        y = nets[i.model].trunk(_enc(torch.cat([dl, torch.linalg.cross(ol, dl)], 1), 8))[1]
        p = torch.sigmoid(y[:, 1])
        D = i.s * (tp - y[:, 0].clamp(-1, 1))
        D = torch.where((p > 0.8) & (D > 0), D, math.inf)
        f = (((p >= 0.2) & (p <= 0.8)) | ((ol * ol).sum(1) < 1)).nonzero()[:, 0]
        A, Df = _march(fields[i.model], ol[f], dl[f], a[f], b[f], 128)
        D[f] = torch.where(A >= 0.5, i.s * Df, math.inf)
        near = D < best[at]
        best[at], who[at] = torch.where(near, D, best[at]), torch.where(near, k, who[at])
    for k, i in enumerate(S.insts):  # secant refinement of the winners
        at = (who == k).nonzero()[:, 0]
        ol, dl = _local(i, o[at], d[at])
        fn = lambda t: fields[i.model].surface(ol + (t / i.s)[:, None] * dl)  # noqa: E731, B023
        D, h = best[at], 0.05 * i.s
        t0, t1, out = D - h, D + h, D.clone()
        f0, f1 = fn(t0), fn(t1)
        live = (f0 < 0) & (f1 >= 0)
        for _ in range(3):
            live = live & (f1 != f0)
            tn = torch.where(live, t1 - f1 * (t1 - t0) / torch.where(f1 != f0, f1 - f0, 1.0), t1)
            live = live & (tn >= D - 2 * h) & (tn <= D + 2 * h)
            out = torch.where(live, tn, out)
            f2 = fn(tn)
            t0, f0 = torch.where(live, t1, t0), torch.where(live, f1, f0)
            t1, f1 = torch.where(live, tn, t1), torch.where(live, f2, f1)
        best[at] = out
    return dict(depth=best, ident=None)


def _exact_train(case, seed):
    st = _prepare_train(case, seed)
    W, b = [_t(w).requires_grad_() for w in st.W], [_t(x).requires_grad_() for x in st.b]
    o, d, alpha, B = st.o.double(), st.d.double(), st.hit.double(), case["batch"]
    tp = -(o * d).sum(1)
    mu = torch.where(alpha > 0, tp - st.depth.double(), 0.0)
    F = torch.nn.functional
    if case["form"] == "line":
        h = _enc(torch.cat([d, torch.linalg.cross(o, d)], 1), 8)
        for w, x in zip(W[:-1], b[:-1]):
            h = torch.relu(F.linear(h, w, x))
        y = F.linear(h, W[-1], b[-1])
        fit = (alpha * (y[:, 0] - mu) ** 2).sum() / B
        bce = F.binary_cross_entropy_with_logits(y[:, 1], alpha)
    else:
        x = [o + tp[:, None] * d + ((2 * k + 1) / 16.0 - 1.0) * d for k in range(16)]
        h = torch.relu(F.linear(torch.cat([_enc(p, 10) for p in x], 1), W[0], b[0]))
        for k in range(16):
            h = h + torch.relu(F.linear(torch.relu(F.linear(h, W[1 + 2 * k], b[1 + 2 * k])), W[2 + 2 * k], b[2 + 2 * k]))
        y = F.linear(h, W[-1], b[-1])
        u = 64 * (mu + 1) / 2
        c = u.floor().clamp(0, 63)
        f = (128 * (u - c)).floor().clamp(0, 127)
        fit = 0.0
        for z, at, n in ((y[:, 1:65], c, 64), (y[:, 65:], f, 128)):
            fit = fit + (alpha[:, None] * F.binary_cross_entropy_with_logits(z, F.one_hot(at.long(), n).double(),
                                                                             reduction="none")).sum() / (n * B)
        bce = F.binary_cross_entropy_with_logits(y[:, 0], alpha)
    loss = fit + 0.1 * bce
    loss.backward()
    new = lambda p: (p - 5e-4 * p.grad / (p.grad.abs() + 1e-8)).detach()  # noqa: E731  (the first Adam step)
    group = lambda v: [v[0], torch.stack(v[1:-1]), v[-1]]  # noqa: E731
    return dict(loss=torch.stack([loss, fit, bce]).detach(), W=group([new(p) for p in W]), b=group([new(p) for p in b]),
                gW=group([p.grad for p in W]), gb=group([p.grad for p in b]))
