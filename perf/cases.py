"""Workloads of the framework's public entry points over the range of sizes that they serve.

listed() names twelve of them, from a coarse-stage render of a few thousand points to a whole view of
several million; draw(rng) makes another one of the same ranges.  prepare(case, seed) holds what a user's
program has on the GPU before the call, run(state) is one pass through the public entry points, work(case)
the bytes and operations that pass cannot do without, and exact(case, seed) the same outputs in 64 bits
from plain torch.

The scenes are the synthetic stand-ins of the repository's benchmark, drawn on the GPU: Gaussian-blob
density logits, normal feature grids, pinhole rays around a box, Bernoulli-thinned midpoint samples, and
for unbounded scenes rays inside the unit ball with disparity-linear samples.
"""
import math

import torch

from paper_2206_05085_amd import autograd, ops, proposal
from paper_2206_05085_amd.step import TrainStep

DEV = "cuda"
F32, F64 = torch.float32, torch.float64
BG = (1.0, 1.0, 1.0)
BOX = ((-1.0, -1.0, -1.0), (1.0, 1.0, 1.0))
HIDDEN, N_FREQ, N_CODE = 128, 4, 27


# ------------------------------------------------------------------------------- cases


def listed():
    return [
        # coarse stage of a bounded scene: density and colour grid, 1024 rays, forward and backward
        dict(name="coarse_render", kind="render_grid", rays=1024, per_ray=128, grid=32, live=1.0),
        # fine-stage rendering under autograd: per-sample colours in, their gradients out
        dict(name="fine_render", kind="render_samples", rays=8192, per_ray=256, grid=160, live=0.6),
        # the training step's render of an unbounded scene: contracted lookups, long ragged rays,
        # loss gradient and density gradient
        dict(name="unbounded_render", kind="render_unbounded", rays=8192, per_ray=280, grid=320),
        # feature lookup of the fine stage and its gradient
        dict(name="features", kind="lookup", rays=8192, per_ray=256, grid=160, channels=12, live=0.6),
        # colour head on one small batch (a few rays: what a preview or a unit of a small scene asks for)
        dict(name="head_small", kind="head", rays=96, per_ray=48, live=0.6),
        # colour head of the fine stage, forward and backward, FP32-grade
        dict(name="head", kind="head", rays=8192, per_ray=256, live=0.6),
        # the cheaper head with the lookup inside it, on a batch thinned by the occupancy mask
        dict(name="head_half", kind="head_half", rays=8192, per_ray=160, grid=160, live=0.5),
        # total variation added into a feature gradient, then the skipping Adam step
        dict(name="grid_update", kind="grid_update", grid=160, channels=12, touched=0.5, dense=True),
        # a training batch made on the GPU from rays and an occupancy mask
        dict(name="sampler", kind="sampler", rays=8192, grid=160, active=0.4),
        # learned sample placement: coarse pass, network, guarded fine batch
        dict(name="proposal", kind="proposal", rays=8192, grid=160, train=False),
        # one view's worth of rays, forward only, stopped at the paper's transmittance
        dict(name="view", kind="view", rays=32768, per_ray=256, grid=160, live=0.6),
        # one whole training iteration on a new batch: bind and step
        dict(name="train_step", kind="train_step", rays=8192, per_ray=256, grid=160, live=0.6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = _draw(rng)
    if "live" in c:  # as many points as the largest listed case of the kind, or a little over
        most = {"view": 5000000, "lookup": 2000000, "render_samples": 2000000, "head_half": 1000000}.get(c["kind"], 1250000)
        c["rays"] = max(32, min(c["rays"], int(most / (c["per_ray"] * c["live"]))))
    return c


def _draw(rng):
    kind = rng.choice(["render_grid", "render_samples", "render_unbounded", "lookup", "head", "head_half",
                       "grid_update", "sampler", "proposal", "view", "train_step"])
    live = round(rng.uniform(0.2, 1.0), 2)
    if kind == "render_grid":
        return dict(kind=kind, rays=_log(rng, 64, 8192), per_ray=rng.randint(16, 200), grid=rng.randint(16, 120), live=live)
    if kind == "render_samples":
        return dict(kind=kind, rays=_log(rng, 64, 16384), per_ray=rng.randint(32, 300), grid=rng.randint(48, 160), live=live)
    if kind == "render_unbounded":
        return dict(kind=kind, rays=_log(rng, 256, 8192), per_ray=rng.randint(64, 280), grid=rng.randint(96, 320))
    if kind == "lookup":
        return dict(kind=kind, rays=_log(rng, 64, 16384), per_ray=rng.randint(32, 256), grid=rng.randint(48, 160),
                    channels=rng.choice([1, 3, 4, 6, 8, 12, 12]), live=live)
    if kind == "head":
        return dict(kind=kind, rays=_log(rng, 48, 12000), per_ray=rng.randint(32, 256), live=live)
    if kind == "head_half":
        return dict(kind=kind, rays=_log(rng, 96, 12000), per_ray=rng.randint(32, 256), grid=rng.randint(48, 160), live=live)
    if kind == "grid_update":
        return dict(kind=kind, grid=rng.randint(24, 170), channels=rng.choice([1, 3, 12, 12]),
                    touched=round(rng.uniform(0.05, 0.9), 2), dense=rng.random() < 0.5)
    if kind == "sampler":
        return dict(kind=kind, rays=_log(rng, 64, 32768), grid=rng.randint(64, 200), active=round(rng.uniform(0.05, 1.0), 2))
    if kind == "proposal":
        return dict(kind=kind, rays=_log(rng, 256, 16384), grid=rng.randint(64, 160), train=rng.random() < 0.5)
    if kind == "view":
        return dict(kind=kind, rays=_log(rng, 512, 32000), per_ray=rng.randint(48, 256), grid=rng.randint(64, 160), live=live)
    return dict(kind="train_step", rays=_log(rng, 256, 8192), per_ray=rng.randint(48, 256), grid=rng.randint(64, 160), live=live)


# ------------------------------------------------------------------------------ inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _rand(g, *shape, dtype=F32):
    return torch.rand(*shape, generator=g, device=DEV, dtype=dtype)


def _blobs(g, n, lo, hi):
    """Blob term of the density logits: 8 Gaussians, amplitude 6..14, width 0.05..0.2."""
    ax = torch.linspace(lo, hi, n, device=DEV)
    mu, sd, amp = _rand(g, 8, 3) * 1.2 - 0.6, 0.05 + 0.15 * _rand(g, 8), 6.0 + 8.0 * _rand(g, 8)
    e = torch.exp(-((ax[None, None, :] - mu[:, :, None]) ** 2) / (2 * sd[:, None, None] ** 2))
    return torch.einsum("b,bx,by,bz->xyz", amp, e[:, 0], e[:, 1], e[:, 2])


def _density(g, n, lo=-1.0, hi=1.0, cleared=False):
    blob, noise = _blobs(g, n, lo, hi), _randn(g, n, n, n)
    d = torch.where(blob >= 1.0, blob + noise, torch.full_like(noise, -20.0)) if cleared else blob + noise
    return d.unsqueeze(-1).contiguous()


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _pinhole(g, R):
    """Random pixels of 100 cameras (800 x 800, 40 degrees) on a sphere of radius 4 that look at the
    origin: origins, unit directions and the box interval (t_far = t_near = 0 for a miss), 64 bits.
    Of the R rays 78 in a hundred hit the box, as of any many such pixels."""
    n = 4 * R + 400
    cams = 4.0 * _unit(torch.randn(100, 3, generator=g, device=DEV, dtype=F64))
    focal = 400.0 / math.tan(math.radians(20.0))
    cid = torch.randint(0, 100, (n,), generator=g, device=DEV)
    px = torch.randint(0, 800, (2, n), generator=g, device=DEV).to(F64) + 0.5
    fwd = _unit(-cams)
    up = torch.tensor([0.0, 0.0, 1.0], device=DEV, dtype=F64).expand(100, 3)
    right = _unit(torch.linalg.cross(fwd, up))
    down = torch.linalg.cross(fwd, right)
    x, y = (px - 400.0) / focal
    d = _unit(x[:, None] * right[cid] + y[:, None] * down[cid] + fwd[cid])
    o = cams[cid]
    t0, t1 = (-1.0 - o) / d, (1.0 - o) / d
    tn = torch.minimum(t0, t1).amax(1).clamp(min=0.0)
    tf = torch.maximum(t0, t1).amin(1)
    hit = tf > tn + 1e-9
    at = torch.arange(n, device=DEV)
    pick = torch.cat([at[hit][:_hits(R)], at[~hit][:R - _hits(R)]])
    pick = pick[torch.randperm(R, generator=g, device=DEV)]
    o, d, tn, tf, hit = (t[pick] for t in (o, d, tn, tf, hit))
    return o, d, torch.where(hit, tn, 0.0), torch.where(hit, tf, 0.0), hit


def _hits(R):
    return int(round(0.78 * R))


def _ragged(live, cols):
    offs = torch.zeros(live.shape[0] + 1, dtype=torch.int32, device=DEV)
    offs[1:] = live.sum(1).cumsum(0).to(torch.int32)
    return offs, [c.expand(live.shape + c.shape[2:])[live].to(F32).contiguous() for c in cols]


def _batch(g, R, N, grid, live):
    """N midpoint samples per ray between its box entry and exit, thinned as an occupancy mask does:
    each ray keeps its own random share, `live` of all of them stay.  Batch, float32 directions."""
    o, d, tn, tf, hit = _pinhole(g, R)
    k = torch.arange(N, device=DEV, dtype=F64)
    step = ((tf - tn) / N)[:, None]
    t = tn[:, None] + (k + 0.5) * step
    keep = hit[:, None].expand(R, N)
    if live < 1.0:
        half = min(0.4, live, 1.0 - live)
        share = live + half * (2.0 * _rand(g, R, 1) - 1.0)
        score = torch.where(keep, _rand(g, R, N, dtype=F64) / share.clamp(min=0.01), 1e9).reshape(-1)
        order = score.argsort(stable=True)[:_samples(dict(kind="", rays=R, per_ray=N, live=live))]
        keep = torch.zeros(R * N, dtype=torch.bool, device=DEV).index_fill_(0, order, True).view(R, N)
    xyz = o[:, None, :] + t[..., None] * d[:, None, :]
    offs, (xyz, delta, sm, sl) = _ragged(keep, [xyz, step * (grid - 1) / 2.0, ((k + 0.5) / N)[None],
                                                torch.full((1, 1), 1.0 / N, device=DEV, dtype=F64)])
    return ops.SampleBatch(offs, xyz, delta, sm, sl, R, xyz.shape[0]), d.to(F32).contiguous()


def _contract(x, b=1.0):
    n = x.abs().amax(-1, keepdim=True)
    return x * torch.where(n <= 1.0, 1.0, (1.0 + b - b / n.clamp(min=1.0)) / n.clamp(min=1.0))


def _unbounded_batch(g, R, per_ray, grid):
    """Rays from a sphere of radius 0.9 into the unit ball; log-normal lengths around per_ray in
    [32, 1024], jittered intervals, s linear in disparity on [0.05, 1000], world points."""
    o = 0.9 * _unit(torch.randn(R, 3, generator=g, device=DEV, dtype=F64))
    aim = _rand(g, R, 1, dtype=F64) ** (1.0 / 3.0) * _unit(torch.randn(R, 3, generator=g, device=DEV, dtype=F64))
    d = _unit(aim - o)
    n = (math.log(0.9 * per_ray) + 0.6 * torch.randn(R, generator=g, device=DEV, dtype=F64)).exp().round().clamp(32, 1024)
    over = _samples(dict(kind="render_unbounded", rays=R, per_ray=per_ray)) - int(n.sum().item())
    n = (n + over // R + (torch.arange(R, device=DEV) < over % R)).clamp(min=1.0)
    n[n.argmax()] += _samples(dict(kind="render_unbounded", rays=R, per_ray=per_ray)) - n.sum()
    top = int(n.max().item())
    j = torch.arange(top + 1, device=DEV, dtype=F64)[None]
    edge = (j + 0.8 * _rand(g, R, top + 1, dtype=F64) - 0.4) / n[:, None]
    edge = torch.where(j <= 0, 0.0, torch.where(j >= n[:, None], 1.0, edge))
    lo, hi = edge[:, :-1], edge[:, 1:]

    def at(s):
        return o[:, None, :] + (1.0 / ((1.0 - s) / 0.05 + s / 1e3))[..., None] * d[:, None, :]

    delta = (_contract(at(hi)) - _contract(at(lo))).norm(dim=-1) * (grid - 1) / 4.0
    keep = j[:, :-1] < n[:, None]
    offs, (xyz, delta, sm, sl) = _ragged(keep, [at(0.5 * (lo + hi)), delta, 0.5 * (lo + hi), hi - lo])
    return ops.SampleBatch(offs, xyz, delta, sm, sl, R, xyz.shape[0]), d.to(F32).contiguous()


def _head_weights(g, channels=12):
    sizes = [channels + N_CODE, HIDDEN, HIDDEN, 3]
    W = [_randn(g, o, i) / math.sqrt(i) for i, o in zip(sizes[:-1], sizes[1:])]
    return W, [0.1 * _randn(g, o) for o in sizes[1:]]


def _moments(g, p, scale):
    """Adam moments of a run that has gone on for a while with gradients of size `scale`."""
    m = scale * 0.3 * _randn(g, *p.shape)
    return m, scale * scale * (0.2 + _rand(g, *p.shape)) + m * m


def _inputs(c, seed):
    """Everything prepare() and exact() share, made from the case and the seed alone."""
    g, kind, s = _gen(seed), c["kind"], {}
    if kind in ("render_grid", "render_samples", "head", "head_half", "lookup", "view", "train_step"):
        s["batch"], s["dirs"] = _batch(g, c["rays"], c["per_ray"], c.get("grid", 160), c["live"])
    elif kind == "render_unbounded":
        s["batch"], s["dirs"] = _unbounded_batch(g, c["rays"], c["per_ray"], c["grid"])
    if "batch" in s:
        S, R, n = s["batch"].n_samples, c["rays"], c.get("grid")
    if kind in ("render_grid", "render_samples"):
        s["density"] = _density(g, n)
        s["colour"] = _rand(g, n, n, n, 3) if kind == "render_grid" else _rand(g, S, 3)
        s["up"] = [_randn(g, R, 3) / R, _randn(g, R) / R, _rand(g, R) * 0.01 / R]
    elif kind == "render_unbounded":
        s["density"], s["colour"], s["target"] = _density(g, n, -2.0, 2.0), _rand(g, S, 3), _rand(g, R, 3)
    elif kind == "lookup":
        s["grid"], s["up"] = _randn(g, n, n, n, c["channels"]), _randn(g, S, c["channels"]) / c["rays"]
    elif kind == "head":
        s["feat"], s["up"] = _randn(g, S, 12), _randn(g, S, 3) / c["rays"]
        s["W"], s["b"] = _head_weights(g)
    elif kind == "head_half":
        s["grid"], s["up"] = _randn(g, n, n, n, 12), _randn(g, S, 3) / c["rays"]
        s["W"], s["b"] = _head_weights(g)
    elif kind == "grid_update":
        n, C = c["grid"], c["channels"]
        s["p"] = _randn(g, n, n, n, C)
        hot = _rand(g, n, n, n // 8 + 1).repeat_interleave(8, 2)[:, :, :n, None] < c["touched"]  # runs along z, as rays leave
        s["g"] = torch.where(hot, 1e-6 * _randn(g, n, n, n, C), 0.0)
        s["m"], s["v"] = _moments(g, s["p"], 1e-6)
    elif kind == "sampler":
        o, d = _pinhole(g, c["rays"])[:2]
        s["rays"] = o.to(F32).contiguous(), d.to(F32).contiguous()
        n = c["grid"]
        blob = _blobs(g, n, -1.0, 1.0)
        cut = blob.flatten()[:: max(1, n ** 3 // 1000000)].quantile(1.0 - c["active"]) if c["active"] < 1.0 else -1.0
        s["mask"] = (blob >= cut).to(torch.uint8).contiguous()
    elif kind == "proposal":
        o, d, tn, tf, _ = _pinhole(g, c["rays"])
        s["rays"] = [t.to(F32).contiguous() for t in (o, d, tn, tf)]
        s["density"] = _density(g, c["grid"], cleared=True)
        s["W"] = [_randn(g, 64, 64) / 8.0 for _ in range(4)]
        s["b"] = [0.05 * _randn(g, 64) for _ in range(4)]
        t = _rand(g, c["rays"], 64) ** 8
        s["target"] = (t / t.sum(1, keepdim=True)).contiguous()
    elif kind in ("view", "train_step"):
        s["density"], s["grid"] = _density(g, n), _randn(g, n, n, n, 12)
        s["W"], s["b"] = _head_weights(g)
        s["target"] = _rand(g, R, 3)
        if kind == "train_step":
            flat = torch.cat([t.reshape(-1) for t in s["W"] + s["b"]])
            s["moments"] = [_moments(g, p, e) for p, e in ((s["density"], 1e-5), (s["grid"], 1e-7), (flat, 1e-4))]
    return s


# --------------------------------------------------------------------------------- run


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    s["case"], s["shift"] = c, ops.act_shift()
    kind = c["kind"]
    if kind in ("render_grid", "render_samples"):
        s["density"].requires_grad_()
        s["colour"].requires_grad_()
    elif kind == "render_unbounded":
        s["grad"] = torch.zeros_like(s["density"])
        s["dg"] = ops.DeviceGrid(s["density"], (-2.0,) * 3, (2.0,) * 3, grad=s["grad"], warp=ops.WARP_CONTRACT_INF)
        b = s["batch"]
        s["bins"] = torch.empty(ops.bin_workspace_size(s["dg"], b.n_samples), dtype=torch.uint8, device=DEV)
        s["state"] = torch.empty(ops.render_state_size(b.n_rays, b.n_samples), dtype=torch.uint8, device=DEV)
        s["g_raw"] = torch.empty(b.n_samples, device=DEV)
    elif kind == "lookup":
        s["grid"].requires_grad_()
    elif kind == "head":
        s["leaves"] = [t.requires_grad_() for t in [s["feat"]] + s["W"] + s["b"]]
    elif kind in ("head_half", "view"):
        half = kind == "head_half"
        s["fg"] = ops.DeviceGrid(s["grid"], *BOX)
        gW, gb = ([torch.zeros_like(t) for t in s["W"]], [torch.zeros_like(t) for t in s["b"]]) if half else (None, None)
        s["mlp"] = ops.MLPParams(s["W"], s["b"], gW, gb, precision=ops.MLP_F16 if half else ops.MLP_SPLIT_F16)
        b = s["batch"]
        s["ws"] = torch.empty(ops.mlp_workspace_size(s["mlp"], b.n_rays, b.n_samples), dtype=torch.uint8, device=DEV)
        if half:
            s["feat"] = torch.empty(b.n_samples, 12, device=DEV)
        else:
            s["dg"] = ops.DeviceGrid(s["density"], *BOX)
    elif kind == "grid_update":
        s["dg"] = ops.DeviceGrid(s["p"], *BOX, grad=s["g"])
    elif kind == "sampler":
        voxel = 2.0 / (c["grid"] - 1)
        s["spec"] = ops.SamplerSpec(*BOX, step=0.5 * voxel, voxel=voxel, mask=s["mask"])
        cap = c["rays"] * 2 * c["grid"]  # a batch's buffers, large enough for any mask
        s["out"] = ops.SampleBatch(None, torch.zeros(cap, 3, device=DEV), *(torch.zeros(cap, device=DEV) for _ in range(3)),
                                   c["rays"], cap)
    elif kind == "proposal":
        s["dg"] = ops.DeviceGrid(s["density"], *BOX)
        s["net"] = proposal.ProposalNet(s["W"], s["b"])
        s["rb"] = ops.RayBatch(*s["rays"])
        cap = c["rays"] * (64 * 4 + 32)  # the fine batch's buffers: at most 4 in each bin, 32 more
        s["fine"] = torch.zeros(cap, 3, device=DEV), *(torch.zeros(cap, device=DEV) for _ in range(3))
    elif kind == "train_step":
        st = TrainStep(s["density"], BOX, feat=s["grid"], mlp=(s["W"], s["b"]))
        for d, (m, v) in zip((st.density, st.feat, st.mlp_flat), s.pop("moments")):
            d["m"], d["v"] = m, v
        st.t_dev.fill_(1000)  # resumed from a checkpoint of step 1000
        s["step"] = st
    return s


def run(state):
    s, c = state, state["case"]
    kind, b = c["kind"], s.get("batch")
    if kind in ("render_grid", "render_samples"):
        out = autograd.render(s["density"], s["colour"], b, BOX, grid_color=kind == "render_grid", act_shift=s["shift"], bg=BG)
        return list(out) + list(torch.autograd.grad(out, [s["density"], s["colour"]], s["up"]))
    if kind == "render_unbounded":
        rgb, T, dist, _, g_rgb = ops.render_train(b, s["dg"], None, s["colour"], s["target"], 0.01, act_shift_=s["shift"],
                                                  bg=BG, state=s["state"], grad_sample_density=s["g_raw"])
        s["grad"].zero_()
        ops.bin_samples(s["dg"], b.xyz, ws=s["bins"])
        ops.grid_scatter_binned(s["dg"], b.xyz, s["g_raw"], s["bins"])
        return [rgb, T, dist, g_rgb, s["g_raw"], s["grad"]]
    if kind == "lookup":
        out = autograd.gather(s["grid"], b.xyz, BOX)
        return [out, torch.autograd.grad(out, s["grid"], s["up"])[0]]
    if kind == "head":
        rgb = autograd.color_mlp(s["feat"], s["W"], s["b"], b.ray_offsets, s["dirs"], N_FREQ)
        return [rgb] + list(torch.autograd.grad(rgb, s["leaves"], s["up"]))
    if kind == "head_half":
        m = s["mlp"]
        rgb = ops.mlp_forward_gather(m, b.ray_offsets, s["dirs"], s["fg"], b.xyz, feat_out=s["feat"], ws=s["ws"])
        for t in m.gW + m.gb:
            t.zero_()
        g = ops.mlp_backward(m, b.ray_offsets, s["dirs"], s["feat"], s["up"], ws=s["ws"], prepared=True)
        return [rgb, s["feat"], g] + m.gW + m.gb
    if kind == "grid_update":
        ops.tv_add_grad(s["dg"], 1e-6, 1.0, c["dense"])
        ops.grid_adam_step(s["p"], s["g"], s["m"], s["v"], lr=0.1, step=1000)
        return [s["p"], s["g"], s["m"], s["v"]]
    if kind == "sampler":
        offs, out = ops.sample_count(s["spec"], *s["rays"]), s["out"]
        ops.sample_emit(s["spec"], *s["rays"], offs, out.n_samples, out=out)
        return [offs, out.xyz, out.delta, out.s_mid, out.s_len]
    if kind == "proposal":
        voxel = 2.0 / (c["grid"] - 1)
        feat, w = proposal.coarse(s["rb"], s["dg"], voxel, s["shift"])
        if c["train"]:
            loss = s["net"].train_step(feat, s["target"])
            return [feat, w, loss, s["net"].flat, s["net"].m, s["net"].v]
        logits, prob, H = s["net"].forward(feat)
        offs, counts = ops.resample_guarded_offsets(s["rb"], prob, w, H, float("inf"))
        ops.resample_guarded(s["rb"], offs, counts, s["fine"][1].numel(), voxel, out=s["fine"])
        return [feat, w, logits, prob, H, offs, counts] + list(s["fine"])
    if kind == "view":
        rgb_s = ops.mlp_forward_gather(s["mlp"], b.ray_offsets, s["dirs"], s["fg"], b.xyz, ws=s["ws"])
        rgb, T, _, _ = ops.render_forward(b, s["dg"], None, rgb_s, act_shift_=s["shift"], halt_T=1e-3, bg=BG, want_dist=False)
        return [rgb_s, rgb, T]
    st = s["step"]
    st.bind(b, s["dirs"], s["target"])
    st.step()
    return [st.rgb, st.T, st.dist, st.loss, [[d["p"], d["m"], d["v"]] for d in (st.density, st.feat, st.mlp_flat)]]


# -------------------------------------------------------------------------------- work


def _samples(c):
    """Samples of a case's batch."""
    if c["kind"] == "render_unbounded":
        return c["rays"] * c["per_ray"]
    return int(round(_hits(c["rays"]) * c["per_ray"] * c.get("live", 1.0)))


def work(case):
    c, kind, R = case, case["kind"], case.get("rays", 0)
    S, V = float(_samples(c) if "per_ray" in c else 0), float(c.get("grid", 0)) ** 3
    U = V * (1.0 - math.exp(-3.0 * S / V)) if V else 0.0  # touched vertices: about 3 new corners a sample
    fwd, bwd = 43520.0 * S, 123648.0 * S  # colour head: forward; recompute and gradients
    ray, smp = 40.0 * R, 24.0 * S
    if kind == "render_grid":
        return {"bytes": smp + 2 * ray + 16 * U + 16 * V, "flops": 400.0 * S}
    if kind == "render_samples":
        return {"bytes": smp + 24 * S + 2 * ray + 4 * U + 4 * V, "flops": 250.0 * S}
    if kind == "render_unbounded":
        return {"bytes": smp + 28 * S + 2 * ray + 4 * U + 4 * V, "flops": 300.0 * S}
    if kind == "lookup":
        C = c["channels"]
        return {"bytes": S * (12 + 8 * C) + 4 * C * (U + V), "flops": 32.0 * C * S}
    if kind == "head":
        return {"bytes": S * (48 + 12 + 12 + 48) + 20 * R, "flops": fwd + bwd}
    if kind == "head_half":
        return {"bytes": S * (12 + 48 + 12 + 12 + 48) + 48 * U + 20 * R, "flops": fwd + bwd}
    if kind == "grid_update":
        N, t = V * c["channels"], 1.0 if c["dense"] else c["touched"]
        return {"bytes": 4 * N * (1 + 7 * t), "flops": 30.0 * N * t}
    if kind == "sampler":
        return {"bytes": 28 * R + V + 24 * 0.6 * R * c["grid"] * c["active"], "flops": 30.0 * 1.6 * R * c["grid"]}
    if kind == "proposal":
        per_ray = 64 * 8 + 60
        return {"bytes": R * per_ray * (1 if c["train"] else 3) + 4 * V * (1 - math.exp(-150.0 * R / V)),
                "flops": R * (64 * 200 + 32768 * (3 if c["train"] else 1))}
    if kind == "view":
        return {"bytes": smp + 12 * S + ray + 52 * U, "flops": fwd + 250 * S}
    # forward, backward, and Adam on the touched vertices (parameters and moments read and written)
    return {"bytes": smp + 2 * ray + 52 * U + 24 * 13 * U, "flops": fwd + bwd + 1000.0 * S}


# ------------------------------------------------------------------- the same in 64 bits


def _interp(grid, xyz, lo, hi, warp=False):
    """Trilinear values of a vertex grid [nx,ny,nz,C] (64 bits) at xyz, clamped to the box."""
    x = xyz.to(F64)
    x = _contract(x) if warp else x
    n = grid.shape[0]
    u = ((x - lo) * ((n - 1) / (hi - lo))).clamp(0, n - 1)
    i = u.floor().clamp(max=n - 2)
    f = u - i
    i = i.long()
    flat, out = grid.reshape(-1, grid.shape[-1]), 0.0
    for k in range(8):
        d = [(k >> 2) & 1, (k >> 1) & 1, k & 1]
        w = 1.0
        for a in range(3):
            w = w * (f[:, a] if d[a] else 1.0 - f[:, a])
        out = out + w[:, None] * flat[((i[:, 0] + d[0]) * n + i[:, 1] + d[1]) * n + i[:, 2] + d[2]]
    return out


def _composite(batch, raw, rgb_s, shift, halt=0.0):
    """Colour, final transmittance and distortion of each ray, and rows of per-sample values."""
    R = batch.n_rays
    offs = batch.ray_offsets.long()
    ln = offs[1:] - offs[:-1]
    N = max(1, int(ln.max().item()))
    ray = torch.repeat_interleave(torch.arange(R, device=DEV), ln)
    at = ray * N + torch.arange(batch.n_samples, device=DEV) - offs[ray]

    def rows(v):
        return torch.zeros((R * N,) + v.shape[1:], device=DEV, dtype=F64).index_copy(0, at, v.to(F64)).view((R, N) + v.shape[1:])

    x = rows(torch.nn.functional.softplus(raw + shift) * batch.delta.to(F64))
    run_x = x.cumsum(1)
    T = torch.exp(x - run_x)
    keep = (T >= halt).to(F64)
    w = T * -torch.expm1(-x) * keep
    TN = torch.exp(-(x * keep).sum(1))
    m, l = rows(batch.s_mid), rows(batch.s_len)
    rgb = (w[..., None] * rows(rgb_s)).sum(1) + TN[:, None]
    W, M = w.cumsum(1) - w, (w * m).cumsum(1) - w * m
    dist = (2.0 * w * (m * W - M) + w * w * l / 3.0).sum(1)
    return rgb, TN, dist


def _head64(feat, W, b, dirs, offs):
    ln = (offs[1:] - offs[:-1]).long()
    d = dirs.to(F64)
    code = torch.cat([d] + [torch.sin(d * 2.0 ** q) for q in range(N_FREQ)] + [torch.cos(d * 2.0 ** q) for q in range(N_FREQ)], 1)
    x = torch.cat([feat, torch.repeat_interleave(code, ln, 0)], 1)
    h = torch.relu(x @ W[0].t() + b[0])
    h = torch.relu(h @ W[1].t() + b[1])
    return torch.sigmoid(h @ W[2].t() + b[2])


def _adam64(p, g, m, v, lr, t, skip):
    m1, v1 = 0.9 * m + 0.1 * g, 0.99 * v + 0.01 * g * g
    p1 = p - lr * (m1 / (1 - 0.9 ** t)) / ((v1 / (1 - 0.99 ** t)).sqrt() + 1e-8)
    if not skip:
        return [p1, m1, v1]
    hot = g != 0
    return [torch.where(hot, a, o) for a, o in ((p1, p), (m1, m), (v1, v))]


def _leaf(t):
    return t.detach().to(F64).requires_grad_()


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "sampler":
        return None  # its integers follow float32 decisions, and every other value hangs on them
    s = _inputs(c, seed)
    shift, b = math.log((1 - 1e-4) ** -2.0 - 1.0), s.get("batch")
    if kind in ("render_grid", "render_samples"):
        den, col = _leaf(s["density"]), _leaf(s["colour"])
        rgb_s = _interp(col, b.xyz, -1.0, 1.0) if kind == "render_grid" else col
        out = _composite(b, _interp(den, b.xyz, -1.0, 1.0)[:, 0], rgb_s, shift)
        g = torch.autograd.grad(out, [den, col], [u.to(F64) for u in s["up"]])
        return [t.detach() for t in out + g]
    if kind == "render_unbounded":
        den, col = _leaf(s["density"]), _leaf(s["colour"])
        raw = _interp(den, b.xyz, -2.0, 2.0, warp=True)[:, 0]
        rgb, T, dist = _composite(b, raw, col, shift)
        loss = ((rgb - s["target"]) ** 2).mean() + 0.01 * dist.mean()
        g_col, g_raw, g_den = torch.autograd.grad(loss, [col, raw, den])
        return [rgb.detach(), T.detach(), dist.detach(), g_col, g_raw, g_den]
    if kind == "lookup":
        grid = _leaf(s["grid"])
        out = _interp(grid, b.xyz, -1.0, 1.0)
        return [out.detach(), torch.autograd.grad(out, grid, s["up"].to(F64))[0]]
    if kind == "head":
        leaves = [_leaf(t) for t in [s["feat"]] + s["W"] + s["b"]]
        rgb = _head64(leaves[0], leaves[1:4], leaves[4:], s["dirs"], b.ray_offsets)
        return [rgb.detach()] + list(torch.autograd.grad(rgb, leaves, s["up"].to(F64)))
    if kind == "head_half":
        feat = _interp(s["grid"].to(F64), b.xyz, -1.0, 1.0).requires_grad_()
        leaves = [feat] + [_leaf(t) for t in s["W"] + s["b"]]
        rgb = _head64(feat, leaves[1:4], leaves[4:], s["dirs"], b.ray_offsets)
        g = torch.autograd.grad(rgb, leaves, s["up"].to(F64))
        return [rgb.detach(), feat.detach()] + list(g)
    if kind == "grid_update":
        p, g, m, v = (s[k].to(F64) for k in "pgmv")
        tv = torch.zeros_like(p)
        for a in range(3):
            d = (p.narrow(a, 1, p.shape[a] - 1) - p.narrow(a, 0, p.shape[a] - 1)).clamp(-1.0, 1.0)
            tv.narrow(a, 1, p.shape[a] - 1).add_(d)
            tv.narrow(a, 0, p.shape[a] - 1).sub_(d)
        hot = True if c["dense"] else (g != 0).any(-1, keepdim=True)
        g = g + (2e-6 / p.numel()) * tv * hot
        p, m, v = _adam64(p, g, m, v, 0.1, 1000, True)
        return [p, g, m, v]
    if kind == "proposal":
        o, d, tn, tf = (t.to(F64) for t in s["rays"])
        k = (torch.arange(64, device=DEV, dtype=F64) + 0.5) / 64.0
        t = tn[:, None] + k * (tf - tn)[:, None]
        x = _interp(s["density"].to(F64), (o[:, None] + t[..., None] * d[:, None]).reshape(-1, 3), -1.0, 1.0)[:, 0].view(-1, 64)
        tau = torch.nn.functional.softplus(x + shift) * ((tf - tn) / 64.0 * (c["grid"] - 1) / 2.0)[:, None]
        w = torch.exp(tau - tau.cumsum(1)) * -torch.expm1(-tau)
        # the network rounds its operands to bfloat16, and the placement follows from it: no such values
        return [torch.log1p(w / 1e-4), w] + [None] * (4 if c["train"] else 9)
    den, grid = _leaf(s["density"]), _leaf(s["grid"])
    W, bb = [_leaf(t) for t in s["W"]], [_leaf(t) for t in s["b"]]
    rgb_s = _head64(_interp(grid, b.xyz, -1.0, 1.0), W, bb, s["dirs"], b.ray_offsets)
    rgb, T, dist = _composite(b, _interp(den, b.xyz, -1.0, 1.0)[:, 0], rgb_s, shift, 1e-3 if kind == "view" else 0.0)
    if kind == "view":
        return [rgb_s.detach(), rgb.detach(), T.detach()]
    loss = ((rgb - s["target"]) ** 2).mean() + 0.01 * dist.mean()
    g = torch.autograd.grad(loss, [den, grid] + W + bb)
    flat = [torch.cat([t.reshape(-1) for t in ts]) for ts in (W + bb, g[2:])]
    new = []
    for (p, gr), (m, v), lr, skip in zip(((den, g[0]), (grid, g[1]), flat), s["moments"], (0.1, 0.1, 1e-3), (True, True, False)):
        new.append(_adam64(p.detach(), gr, m.to(F64), v.to(F64), lr, 1001, skip))
    return [rgb.detach(), T.detach(), dist.detach(), loss.detach().reshape(1), new]
