"""The work that users of this framework have it do, as cases to be timed.

A case is a dict of plain values; `kind` names what is called:

  animate     runtime animation: weights MLP, blend, render, status read
  serve       one batch of the animation server (avatars of different sizes)
  autograd    BlendRender under torch autograd, an L2 loss and its gradients
  train       the batched training step of `Trainer`, captured as a graph
  uneven      the batched step over frames of different sizes, from the
              library's entry points, captured as a graph
  render      a batch's render and its adjoint on given blended Gaussians
  blend, blend_grad, mlp, adam, loss    the step's other layers by themselves

Sizes: 2,000 to 100,000 Gaussians, 5 to 40 blendshapes, batches of 1 to 64
frames, images of 128 to 512 pixels a side (square and ragged), the default
tile of 16 pixels with the chunks of 64 and 128 entries that tuning picks.
Values follow the seeded synthetic avatars of `synth`, drawn on the device.

The two training kinds run at learning rates of zero, the first step of a
warm-up ramp: the step does all its work and returns its loss and the
optimiser's moments (and so the gradients), and every pass sees the same
scene, so passes can be repeated and compared.  `adam` covers the update at
the trainer's own rates.
"""
import math

import numpy as np
import torch

from paper_2503_12886_amd import autograd, gbr, serve, synth
from paper_2503_12886_amd.trainer import ADAM_BETAS, ADAM_EPS, StepConfig, Trainer, bases_lr_table, mlp_numel, mlp_pack

D_IN, HIDDEN = synth.THETA_DIM, synth.MLP_HIDDEN
SERVE_NS = "20000,40000,60000,80000,100000,100000,50000,30000"
UNEVEN_RES = [(256, 256), (384, 384), (512, 512)]
ENTRIES_PER_SPLAT = 34        # tile entries a Gaussian is given room for (18 to 26 are met at 512 x 512)
PAIRS_PER_PIXEL = 20          # contributing Gaussians of a pixel, as the benchmark's training batch has
GRAD_STD = 1e-6               # size of a gradient entry under a loss averaged over a batch's pixels


def listed():
    return [
        # one frame of an avatar as it is animated: latency and launches
        dict(name="animate_one", kind="animate", N=50_000, K=20, B=1, W=512, H=512, chunk=64),
        # a full batch of the server: eight avatars of different sizes
        dict(name="serve_batch", kind="serve", ns=SERVE_NS, K=20, W=512, H=512),
        # a small model fitted through torch autograd, one frame per call: the smallest step
        dict(name="autograd_small", kind="autograd", N=2_000, K=8, B=1, W=128, H=128, chunk=64),
        # the benchmark's training step, a few replays in a row as a fit runs them
        dict(name="train_512", kind="train", N=50_000, K=20, B=16, W=512, H=512, chunk=64, loss=1, mesh=False, steps=4),
        # the paper's batch of ten with Gaussians bound to a tracked mesh
        dict(name="train_mesh", kind="train", N=60_000, K=20, B=10, W=512, H=512, chunk=64, loss=1, mesh=True, steps=4),
        # the largest step: 64 frames of three sizes at different distances
        dict(name="train_uneven", kind="uneven", N=100_000, K=20, B=64, chunk=64, sizes=23),
        # a small batch of odd-sized frames, forward and backward, the other chunk
        dict(name="render_ragged", kind="render", N=30_011, B=5, W=333, H=500, chunk=128),
        # the large avatar's blend at twice the usual blendshapes
        dict(name="blend_k40", kind="blend", N=100_000, K=40, B=8),
        # the blend's adjoint by itself (gradients of the bases written out), an odd count
        dict(name="blend_grad", kind="blend_grad", N=60_001, K=20, B=10),
        # the weights network of a batch, forward and backward
        dict(name="mlp_16", kind="mlp", K=20, B=16),
        # the update of the bases with its gradient formed inside
        dict(name="adam_bases", kind="adam", N=50_000, K=20, B=16),
        # the photometric loss and its image gradient over a batch
        dict(name="loss_l1", kind="loss", B=16, W=512, H=512, loss=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["animate", "serve", "autograd", "train", "train", "train", "uneven", "render", "render",
                       "blend", "blend_grad", "mlp", "adam", "loss"])
    c = dict(kind=kind)
    if kind == "serve":
        c.update(ns=",".join(str(_log(rng, 20_000, 100_000)) for _ in range(rng.randint(2, 8))), K=20,
                 W=rng.randint(256, 512), H=rng.randint(256, 512))
        return c
    if kind not in ("mlp", "loss"):
        c["N"] = _log(rng, 2_000, 100_000)
    if kind not in ("render", "loss"):
        c["K"] = rng.randint(5, 40)
    if kind == "uneven":
        c.update(B=_log(rng, 4, 32), chunk=rng.choice([64, 128]), sizes=rng.randrange(1000))
        return c
    c["B"] = 1 if kind == "animate" else _log(rng, 1, 4 if kind == "autograd" else 32 if kind == "blend" else 16)
    if kind in ("animate", "autograd", "train", "render", "loss"):
        c.update(W=_log(rng, 128, 512), H=_log(rng, 128, 512))
    if kind in ("animate", "autograd", "train", "render"):
        c["chunk"] = rng.choice([64, 64, 128])
    if kind in ("train", "loss"):
        c["loss"] = rng.choice([1, 1, 2])
    if kind == "train":
        c.update(mesh=rng.random() < 0.3, steps=rng.randint(1, 4))
    return c


# ---------------------------------------------------------------- inputs
class _Rand:
    """Seeded draws on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.randn(*shape, generator=self.g, device="cuda") * std + mean

    def uniform(self, *shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, generator=self.g, device="cuda") * (hi - lo) + lo


def _scene(r, N, K, surface=False):
    """Bases [K + 1, N, 16] of a synthetic avatar (synth.make_scene; with
    surface, synth.make_tangent_scene: small offsets from a mesh point)."""
    b = torch.zeros(K + 1, N, 16, device="cuda")
    d = r.normal(N, 3)
    d = d / d.norm(dim=1, keepdim=True) * r.uniform(N, 1) ** (1.0 / 3.0)
    b[0, :, 0:3] = d * torch.tensor([0.08, 0.10, 0.09], device="cuda")
    q = r.normal(N, 4)
    b[0, :, 3:7] = q / q.norm(dim=1, keepdim=True)
    b[0, :, 7:10] = r.normal(N, 3, std=0.3, mean=-5.0)
    b[0, :, 10] = r.normal(N)
    b[0, :, 11:14] = r.uniform(N, 3)
    if surface:
        b[0, :, 0:3] = r.normal(N, 3, std=5e-3) * torch.tensor([1.0, 1.0, 0.2], device="cuda")
    if K:
        b[1:, :, :14] = r.normal(K, N, 14, std=1e-3)
    return b


def _perturbed(r, bases, pos_std):
    """A fit's starting point: the base model with noise (synth.perturb_scene)."""
    out = bases.clone()
    N = bases.shape[1]
    out[0, :, 0:3] += r.normal(N, 3, std=pos_std)
    out[0, :, 3:7] += r.normal(N, 4, std=0.05)
    out[0, :, 7:10] += r.normal(N, 3, std=0.1)
    out[0, :, 10] += r.normal(N, std=0.3)
    out[0, :, 11:14] += r.normal(N, 3, std=0.05)
    return out


def _blended(r, N, B):
    """Blended Gaussians [B, N, 16]: one avatar under B expressions."""
    raw = _scene(r, N, 0)[0].expand(B, N, 16).contiguous()
    raw[:, :, :14] += r.normal(B, N, 14, std=3e-3)
    return raw


def _grads(r, *shape):
    """Gradients of blended Gaussians (the two pad features are zero)."""
    g = r.normal(*shape, std=GRAD_STD)
    g[..., 14:] = 0.0
    return g


def _moments(r, shape):
    """Adam's moments of a fit under way."""
    return r.normal(*shape, std=GRAD_STD), r.uniform(*shape, lo=0.5, hi=1.5) * GRAD_STD ** 2


def _mlp(K, seed):
    return mlp_pack(synth.make_mlp(K=K, seed=seed))


def _cams(c, seed, count=None):
    return synth.make_cameras(count or c["B"], c["W"], c["H"], seed=seed, bg_seed=seed + 1)


def _offsets(N, B):
    return [b * N for b in range(B + 1)]


def _context(cams, splats, chunk, entries=None):
    return gbr.Context(tile=16, chunk=chunk, max_frames=len(cams), max_splats=splats,
                       max_pixels=sum(k.width * k.height for k in cams),
                       max_entries=entries or max(1 << 16, ENTRIES_PER_SPLAT * splats))


def _sized_render(ctx, raw, offsets, cams, images):
    """A first render that leaves the context with room for the batch's tile entries."""
    gbr.gbr_render(ctx, raw, offsets, cams, images)
    st = gbr.gbr_query_status(ctx)
    if st.overflow:
        gbr.gbr_reserve(ctx, st.entries + st.entries // 4 + 4096)


class _State:
    """What a program holds between calls; gives its library handles back."""

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        if getattr(self, "graph", None) is not None:
            gbr.gbr_graph_destroy(self.graph)
        for h in ("trainer", "executor", "ctx"):
            if getattr(self, h, None) is not None:
                getattr(self, h).close()


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, _Rand(seed), seed)


def run(state):
    return state.call(state)


# ---------------------------------------------------------------- animation
def _prepare_animate(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    cams = _cams(c, seed)
    s = _State(call=_run_animate, c=c, cams=cams, offsets=_offsets(N, B), bases=_scene(r, N, K),
               mlp=torch.from_numpy(_mlp(K, seed)).cuda(),
               theta=torch.from_numpy(synth.make_tracking(B, seed=seed)).cuda(),
               psi=torch.zeros(B, K, device="cuda"), raw=torch.zeros(B, N, 16, device="cuda"),
               images=torch.zeros(gbr.image_numel(cams), device="cuda"), ctx=_context(cams, B * N, c["chunk"]))
    gbr.gbr_blend(s.ctx, s.bases, s.psi, s.raw)
    _sized_render(s.ctx, s.raw, s.offsets, cams, s.images)
    return s


def _run_animate(s):
    gbr.gbr_mlp_forward(s.ctx, s.mlp, s.theta, D_IN, HIDDEN, s.c["K"], s.psi)
    gbr.gbr_blend(s.ctx, s.bases, s.psi, s.raw)
    gbr.gbr_render(s.ctx, s.raw, s.offsets, s.cams, s.images)
    gbr.gbr_query_status(s.ctx)          # whether the frame is whole
    return {"psi": s.psi, "images": s.images}


def _prepare_serve(c, r, seed):
    ns = [int(n) for n in c["ns"].split(",")]
    bases = [_scene(r, n, c["K"]).cpu().numpy() for n in ns]
    mlps = [_mlp(c["K"], seed + i) for i in range(len(ns))]
    ex = serve.GpuExecutor(bases, mlps, n_slots=1, max_batch=len(ns), width=c["W"], height=c["H"])
    theta = synth.make_tracking(len(ns), seed=seed)
    cams = _cams(c, seed, len(ns))
    order = np.random.default_rng(seed).permutation(len(ns))
    batch = [serve.Request(rid=i, avatar=int(a), theta=theta[i], cam=cams[i], t_arrival=0.0)
             for i, a in enumerate(order)]
    s = _State(call=_run_serve, executor=ex, batch=batch)
    _run_serve(s)
    return s


def _run_serve(s):
    handle = s.executor.launch(0, s.batch)
    s.executor.finish(handle)
    return {"images": s.executor.slots[0]["images"]}


# ---------------------------------------------------------------- fitting
def _prepare_autograd(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    cams = _cams(c, seed)
    s = _State(call=_run_autograd, cams=cams, bases=_scene(r, N, K).requires_grad_(),
               weights=r.uniform(B, K).requires_grad_(), target=r.uniform(gbr.image_numel(cams)),
               ctx=_context(cams, B * N, c["chunk"]))
    return s


def _run_autograd(s):
    images = autograd.blend_render(s.bases, s.weights, s.cams, s.ctx)
    loss = (images - s.target).square().mean()
    dbases, dweights = torch.autograd.grad(loss, [s.bases, s.weights])
    return {"images": images.detach(), "loss": loss.detach(), "dbases": dbases, "dweights": dweights}


def _prepare_train(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    cfg = StepConfig(N=N, K=K, B=B, width=c["W"], height=c["H"], loss=c["loss"], chunk=c["chunk"])
    bases = _scene(r, N, K, surface=c["mesh"])
    t = Trainer(cfg, bases.cpu().numpy(), _mlp(K, seed))
    verts = None
    if c["mesh"]:
        base, faces, uv = synth.make_head_mesh()
        verts = synth.deform_mesh(base, B, seed=seed)
        t.bind_mesh(faces, uv, *synth.bind_gaussians(faces, base, N, seed=seed), base.shape[0])
    t.set_batch(synth.make_tracking(B, seed=seed), np.zeros(t.targets.numel(), np.float32), _cams(c, seed), verts=verts)
    t.render_targets()                   # the avatar's own frames; the fit starts from a perturbed copy
    torch.cuda.synchronize()
    t.bases.copy_(_perturbed(r, bases, 5e-4 if c["mesh"] else 2e-3))
    t.lr_bases, t.lr_mlp = [0.0] * 32, [0.0] * 32
    torch.cuda.synchronize()
    t.step()                             # sizes the buffers
    for m, v in ((t.bases_m, t.bases_v), (t.mlp_m, t.mlp_v)):
        m0, v0 = _moments(r, m.shape)
        m.copy_(m0)
        v.copy_(v0)
    t.capture()
    return _State(call=_run_train, c=c, trainer=t)


def _run_train(s):
    t = s.trainer
    st = t.run_steps(s.c["steps"])
    return {"loss": st.loss, "entries": st.entries, "images": t.images, "draw": t.draw, "dpsi": t.dpsi,
            "dmlp": t.dmlp, "bases": t.bases, "m": t.bases_m, "v": t.bases_v, "mlp_m": t.mlp_m, "mlp_v": t.mlp_v}


def _prepare_uneven(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    rng = np.random.default_rng(c["sizes"])            # the frames' sizes are the case's, the rest the seed's
    cams = [synth.make_cameras(1, *UNEVEN_RES[rng.integers(3)], seed=seed + b, dist=(0.4, 0.7),
                               bg_seed=seed + 64 + b)[0]
            for b in range(B)]
    npx = sum(k.width * k.height for k in cams)
    bases = _scene(r, N, K)
    m, v = _moments(r, bases.shape)
    f32 = dict(device="cuda", dtype=torch.float32)
    s = _State(call=_run_uneven, cams=cams, offsets=_offsets(N, B), bases=bases, m=m, v=v, weights=r.uniform(B, K),
               targets=r.uniform(3 * npx), raw=torch.empty(B, N, 16, **f32), draw=torch.empty(B, N, 16, **f32),
               images=torch.empty(3 * npx, **f32), dimages=torch.empty(3 * npx, **f32),
               dweights=torch.empty(B, K, **f32), ctx=_context(cams, B * N, c["chunk"]))
    gbr.gbr_blend(s.ctx, s.bases, s.weights, s.raw)
    _sized_render(s.ctx, s.raw, s.offsets, cams, s.images)
    torch.cuda.synchronize()
    s.stream = torch.cuda.Stream()       # a captured step needs a stream of its own
    with torch.cuda.stream(s.stream):
        gbr.gbr_graph_begin(s.ctx, s.stream)
        try:
            gbr.gbr_blend(s.ctx, s.bases, s.weights, s.raw)
            gbr.gbr_render(s.ctx, s.raw, s.offsets, cams, s.images)
            gbr.gbr_loss(s.ctx, s.images, s.targets, 1, s.dimages)
            gbr.gbr_render_backward(s.ctx, s.dimages, s.draw)
            gbr.gbr_blend_backward(s.ctx, s.draw, s.bases, s.weights, None, s.dweights)
            gbr.gbr_blend_adam_step(s.ctx, 0, s.draw, s.weights, s.bases, s.m, s.v, [0.0] * 32, ADAM_BETAS[0],
                                    ADAM_BETAS[1], ADAM_EPS)
        finally:
            s.graph = gbr.gbr_graph_end(s.ctx, s.stream)
    return s


def _run_uneven(s):
    gbr.gbr_graph_launch(s.graph, s.stream)
    st = gbr.gbr_query_status(s.ctx, s.stream)
    return {"loss": st.loss, "entries": st.entries, "images": s.images, "draw": s.draw, "dweights": s.dweights,
            "bases": s.bases, "m": s.m, "v": s.v}


# ---------------------------------------------------------------- single layers
def _prepare_render(c, r, seed):
    N, B = c["N"], c["B"]
    cams = _cams(c, seed)
    n = gbr.image_numel(cams)
    s = _State(call=_run_render, cams=cams, offsets=_offsets(N, B), raw=_blended(r, N, B),
               images=torch.zeros(n, device="cuda"), dimages=r.normal(n, std=1.0 / n),
               draw=torch.zeros(B, N, 16, device="cuda"), ctx=_context(cams, B * N, c["chunk"]))
    _sized_render(s.ctx, s.raw, s.offsets, cams, s.images)
    return s


def _run_render(s):
    gbr.gbr_render(s.ctx, s.raw, s.offsets, s.cams, s.images)
    gbr.gbr_render_backward(s.ctx, s.dimages, s.draw)
    return {"images": s.images, "draw": s.draw}


def _layer_context(B, N):
    """A context for calls that render nothing larger than a pixel."""
    return gbr.Context(max_frames=B, max_splats=B * N, max_pixels=64, max_entries=1024)


def _prepare_blend(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    return _State(call=_run_blend, bases=_scene(r, N, K), weights=r.uniform(B, K, lo=-0.5, hi=1.0),
                  raw=torch.zeros(B, N, 16, device="cuda"), ctx=_layer_context(B, 1))


def _run_blend(s):
    gbr.gbr_blend(s.ctx, s.bases, s.weights, s.raw)
    return s.raw


def _prepare_blend_grad(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    return _State(call=_run_blend_grad, bases=_scene(r, N, K), weights=r.uniform(B, K, lo=-0.5, hi=1.0),
                  draw=_grads(r, B, N, 16), dbases=torch.zeros(K + 1, N, 16, device="cuda"),
                  dweights=torch.zeros(B, K, device="cuda"), ctx=_layer_context(B, N))


def _run_blend_grad(s):
    gbr.gbr_blend_backward(s.ctx, s.draw, s.bases, s.weights, s.dbases, s.dweights)
    return {"dbases": s.dbases, "dweights": s.dweights}


def _prepare_mlp(c, r, seed):
    K, B = c["K"], c["B"]
    params = torch.from_numpy(_mlp(K, seed)).cuda()
    return _State(call=_run_mlp, K=K, params=params, theta=torch.from_numpy(synth.make_tracking(B, seed=seed)).cuda(),
                  psi=torch.zeros(B, K, device="cuda"), dpsi=r.normal(B, K, std=1e-3),
                  dparams=torch.zeros_like(params), ctx=_layer_context(B, 1))


def _run_mlp(s):
    gbr.gbr_mlp_forward(s.ctx, s.params, s.theta, D_IN, HIDDEN, s.K, s.psi)
    gbr.gbr_mlp_backward(s.ctx, s.params, s.dpsi, s.dparams)
    return {"psi": s.psi, "dparams": s.dparams}


def _prepare_adam(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    bases = _scene(r, N, K)
    m, v = _moments(r, bases.shape)
    return _State(call=_run_adam, lr=bases_lr_table(), bases=bases, m=m, v=v, draw=_grads(r, B, N, 16),
                  weights=r.uniform(B, K, lo=-0.5, hi=1.0), ctx=_layer_context(B, N))


def _run_adam(s):
    gbr.gbr_blend_adam_step(s.ctx, 0, s.draw, s.weights, s.bases, s.m, s.v, s.lr, ADAM_BETAS[0], ADAM_BETAS[1],
                            ADAM_EPS)
    return {"bases": s.bases, "m": s.m, "v": s.v}


def _prepare_loss(c, r, seed):
    cams = _cams(c, seed)
    n = gbr.image_numel(cams)
    s = _State(call=_run_loss, loss=c["loss"], images=r.uniform(n), dimages=torch.zeros(n, device="cuda"),
               ctx=_context(cams, c["B"] * 16, 64))
    s.targets = s.images + r.normal(n, std=0.1)
    gbr.gbr_preprocess(s.ctx, _blended(r, 16, c["B"]), _offsets(16, c["B"]), cams)   # the batch's frame sizes
    return s


def _run_loss(s):
    gbr.gbr_loss(s.ctx, s.images, s.targets, s.loss, s.dimages)
    return s.dimages


# ---------------------------------------------------------------- work
def work(case):
    """Bytes and operations of one pass that no implementation can do without."""
    c, kind = case, case["kind"]
    B, N, K = c.get("B", 1), c.get("N", 0), c.get("K", 0)
    px = B * c.get("W", 0) * c.get("H", 0)
    slices, splats = (K + 1) * N * 64, B * N * 64        # the bases; one value per blended Gaussian and feature
    fwd, bwd = 22 * PAIRS_PER_PIXEL, 59 * PAIRS_PER_PIXEL
    mlp = mlp_numel(D_IN, HIDDEN, K)
    if kind == "serve":
        ns = [int(n) for n in c["ns"].split(",")]
        px = len(ns) * c["W"] * c["H"]
        return {"bytes": sum((K + 1) * n * 64 for n in ns) + 4 * mlp * len(ns) + 12 * px,
                "flops": px * fwd + sum(2 * K * n * 14 for n in ns)}
    if kind == "animate":
        return {"bytes": slices + 4 * mlp + 12 * px, "flops": px * fwd + 2 * B * K * N * 14}
    if kind == "autograd":
        return {"bytes": 2 * slices + 24 * px, "flops": px * (fwd + bwd) + 6 * B * K * N * 14}
    if kind == "train":
        return {"bytes": c["steps"] * (6 * slices + 28 * mlp + 24 * px),
                "flops": c["steps"] * (px * (fwd + bwd) + 6 * B * K * N * 14)}
    if kind == "uneven":
        px = B * sum(w * h for w, h in UNEVEN_RES) // len(UNEVEN_RES)
        return {"bytes": 6 * slices + 24 * px, "flops": px * (fwd + bwd) + 6 * B * K * N * 14}
    if kind == "render":
        return {"bytes": 2 * splats + 24 * px, "flops": px * (fwd + bwd)}
    if kind == "blend":
        return {"bytes": slices + splats, "flops": 2 * B * K * N * 14}
    if kind == "blend_grad":
        return {"bytes": 2 * slices + splats, "flops": 4 * B * K * N * 14}
    if kind == "mlp":
        return {"bytes": 8 * mlp, "flops": 6 * B * mlp}
    if kind == "adam":
        return {"bytes": 6 * slices + splats, "flops": (2 * B + 12) * (K + 1) * N * 14}
    return {"bytes": 36 * px, "flops": 6 * px}


# ---------------------------------------------------------------- the same in 64 bits
EXACT_PAIRS = 80_000_000      # (pixel, Gaussian) pairs a plain render goes through


def exact(case, seed):
    f = globals().get("_exact_" + case["kind"])
    return f(case, _Rand(seed), seed) if f else None


def _exact_blend(c, r, seed):
    bases = _scene(r, c["N"], c["K"]).double()
    w = r.uniform(c["B"], c["K"], lo=-0.5, hi=1.0).double()
    return (bases[0].reshape(1, -1) + w @ bases[1:].reshape(c["K"], -1)).reshape(c["B"], c["N"], 16)


def _exact_blend_grad(c, r, seed):
    bases = _scene(r, c["N"], c["K"]).double()
    w = r.uniform(c["B"], c["K"], lo=-0.5, hi=1.0).double()
    d = _grads(r, c["B"], c["N"], 16).double().reshape(c["B"], -1)
    dbases = torch.cat([d.sum(0, keepdim=True), w.t() @ d]).reshape(bases.shape)
    return {"dbases": dbases, "dweights": d @ bases[1:].reshape(c["K"], -1).t()}


def _exact_mlp(c, r, seed):
    K, B = c["K"], c["B"]
    p = torch.from_numpy(_mlp(K, seed)).cuda().double().requires_grad_()
    dims = [(HIDDEN, D_IN), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (K, HIDDEN), (K,)]
    W1, b1, W2, b2, W3, b3 = (x.reshape(d) for x, d in zip(p.split([int(np.prod(d)) for d in dims]), dims))
    x = torch.from_numpy(synth.make_tracking(B, seed=seed)).cuda().double()
    psi = torch.relu(torch.relu(x @ W1.t() + b1) @ W2.t() + b2) @ W3.t() + b3
    dpsi = r.normal(B, K, std=1e-3).double()
    dparams, = torch.autograd.grad((psi * dpsi).sum(), [p])
    return {"psi": psi.detach(), "dparams": dparams}


def _exact_adam(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    bases = _scene(r, N, K).double()
    m, v = (x.double() for x in _moments(r, bases.shape))
    d = _grads(r, B, N, 16).double().reshape(B, -1)
    w = r.uniform(B, K, lo=-0.5, hi=1.0).double()
    g = torch.cat([d.sum(0, keepdim=True), w.t() @ d]).reshape(bases.shape)
    b1, b2 = (float(np.float32(b)) for b in ADAM_BETAS)
    m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
    lr = torch.tensor(bases_lr_table(), device="cuda").double().reshape(2, 16)
    rate = torch.cat([lr[:1], lr[1:].expand(K, 16)]).reshape(K + 1, 1, 16)
    step = rate * (m / (1 - b1)) / (torch.sqrt(v / (1 - b2)) + ADAM_EPS)
    return {"bases": bases - step, "m": m, "v": v}


def _exact_loss(c, r, seed):
    n = 3 * c["B"] * c["W"] * c["H"]
    x = r.uniform(n)
    y = x + r.normal(n, std=0.1)
    d = x.double() - y.double()
    return torch.sign(d) / n if c["loss"] == 1 else 2.0 * d / n


def _plain_image(raw, cam):
    """One frame in 64 bits: activations, projection, and every pixel's
    front-to-back compositing over all Gaussians in depth order."""
    f64 = dict(device=raw.device, dtype=torch.float64)
    R, t = torch.as_tensor(cam.R, **f64), torch.as_tensor(cam.t, **f64)
    p = raw[:, 0:3] @ R.t() + t
    order = torch.sort(p[:, 2].detach().float(), stable=True).indices
    order = order[p[order, 2].detach() > cam.near]
    raw, p = raw[order], p[order]
    x, y, z = p.unbind(1)
    q = raw[:, 3:7] / raw[:, 3:7].norm(dim=1, keepdim=True)
    a, b, c, d = q.unbind(1)
    rot = torch.stack([1 - 2 * (c * c + d * d), 2 * (b * c - a * d), 2 * (b * d + a * c),
                       2 * (b * c + a * d), 1 - 2 * (b * b + d * d), 2 * (c * d - a * b),
                       2 * (b * d - a * c), 2 * (c * d + a * b), 1 - 2 * (b * b + c * c)], 1).reshape(-1, 3, 3)
    M = rot * raw[:, 7:10].exp().unsqueeze(1)
    zero = torch.zeros_like(z)
    J = torch.stack([cam.fx / z, zero, -cam.fx * x / (z * z), zero, cam.fy / z, -cam.fy * y / (z * z)], 1)
    V = (J.reshape(-1, 2, 3) @ R) @ M
    S = V @ V.transpose(1, 2)
    sa, sb, sc = S[:, 0, 0] + 0.3, S[:, 0, 1], S[:, 1, 1] + 0.3
    det = sa * sc - sb * sb
    mx, my = cam.fx * x / z + cam.cx, cam.fy * y / z + cam.cy
    ys, xs = torch.meshgrid(torch.arange(cam.height, **f64) + 0.5, torch.arange(cam.width, **f64) + 0.5, indexing="ij")
    dx, dy = xs.reshape(-1, 1) - mx, ys.reshape(-1, 1) - my
    power = -0.5 * (sc * dx * dx - 2 * sb * dx * dy + sa * dy * dy) / det
    alpha = torch.sigmoid(raw[:, 10]) * power.exp()
    alpha = torch.where(alpha >= 1.0 / 255.0, alpha.clamp(max=0.99), 0.0)
    alpha = torch.where((1 - alpha).cumprod(1) >= 1e-4, alpha, 0.0)      # the pixel stops before that entry
    through = (1 - alpha).cumprod(1)
    front = torch.cat([torch.ones_like(through[:, :1]), through[:, :-1]], 1)
    out = (alpha * front) @ raw[:, 11:14] + through[:, -1:] * torch.as_tensor(cam.bg, **f64)
    return out.t().reshape(3, cam.height, cam.width)


def _exact_autograd(c, r, seed):
    N, K, B = c["N"], c["K"], c["B"]
    if B * N * c["W"] * c["H"] > EXACT_PAIRS:
        return None
    cams = _cams(c, seed)
    bases = _scene(r, N, K).double().requires_grad_()
    weights = r.uniform(B, K).double().requires_grad_()
    target = r.uniform(gbr.image_numel(cams)).double()
    raw = (bases[0].reshape(1, -1) + weights @ bases[1:].reshape(K, -1)).reshape(B, N, 16)
    images = torch.cat([_plain_image(raw[b], k).reshape(-1) for b, k in enumerate(cams)])
    loss = (images - target).square().mean()
    dbases, dweights = torch.autograd.grad(loss, [bases, weights])
    return {"images": images.detach(), "loss": loss.detach(), "dbases": dbases, "dweights": dweights}
