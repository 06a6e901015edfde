"""The work a user of the rasterizer has it do, as cases that can be timed and compared.

Five kinds, each through the public entry points of `paper_2603_27151_amd.raster`:

* ``step``: forward, loss and backward of the workloads' form. Options: the loss (L2, or the
  training loss L1 + D-SSIM), the calls themselves or the autograd function (which also returns
  log p), and whether the forward keeps its fragment log for the backward (``keep``) or the
  backward finds the fragments again, as the training loop does.
* ``render``: forward-only renders of several requests in threshold mode, as the server does.
* ``paper``: assembly of the mesh-colour texture, forward, loss and backward of the paper form;
  the backward with the levels folded in, or the texture's gradient followed by the assembly's.
* ``adam``: one optimiser step over every parameter of a soup.
* ``adapt``: coverage of a batch of views, edge lengths over a sample of views, the plan and the
  rebuilt soup.

Sizes are those of the framework's own workloads; drawn cases spread over the same ranges.
Views look at the origin from a sphere of radius 3. Each case's sizes are independent of the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_27151_amd import raster as R
from paper_2603_27151_amd import workloads as W

FORMS = {"8-16-4": [8, 16, 4], "16-32-32-4": [16, 32, 32, 4], "32-64-64-4": [32, 64, 64, 4]}
BG_KEY = 2 ** 63 - 1


def _sizes(text):
    return [tuple(int(n) for n in s.split("x")) for s in text.split(",")]


def _text(sizes):
    return ",".join("%dx%d" % s for s in sizes)


def listed():
    mixed = [W.BATCHED_RES[int(k)] for k in   # as the batched workload draws them
             "0321113120313210012213220212022031100201001312310200300010030233"]
    burst = [W.SERVING_RES[k] for k in (0, 1, 2, 1, 0, 2, 1, 1, 0, 2, 0, 1, 2, 1, 0, 2)]
    return [
        # the smallest step: a unit test, a debugging session; launches and host work count
        dict(name="step_tiny", kind="step", form="8-16-4", G=4, T=64, soup="box", sizes="128x128", loss="l2",
             api="calls", keep=True),
        # one training view of a small soup
        dict(name="step_single", kind="step", form="16-32-32-4", G=8, T=10_000, soup="ball", sizes="800x800",
             loss="l2", api="calls", keep=True),
        # odd image sizes through the autograd function, with log p, as a user's own torch loop has it
        dict(name="step_odd_autograd", kind="step", form="16-32-32-4", G=8, T=5_000, soup="ball",
             sizes="517x389,641x365", loss="l2", api="autograd", keep=True),
        # the headline: 64 views of uneven resolution in one step
        dict(name="step_batched", kind="step", form="16-32-32-4", G=8, T=50_000, soup="ball",
             sizes=_text([(r, r) for r in mixed]), loss="l2", api="calls", keep=True),
        # the largest step: deep, clustered, the widest decoder
        dict(name="step_large", kind="step", form="32-64-64-4", G=8, T=200_000, soup="blobs",
             sizes=_text([(1920, 1080)] * 16), loss="l2", api="calls", keep=True),
        # one iteration of the training loop: four views, L1 + D-SSIM, no fragment log kept
        dict(name="train_four_views", kind="step", form="16-32-32-4", G=8, T=50_000, soup="ball",
             sizes="800x800,512x512,1024x1024,256x256", loss="l1_ssim", api="calls", keep=False),
        # a lone request at a server: latency
        dict(name="render_one", kind="render", T="20000", sizes="640x360"),
        # a full batch of requests at a busy server: four resident soups, three resolutions
        dict(name="render_burst", kind="render", T=",".join(str(t) for t in W.SERVING_SOUPS), sizes=_text(burst)),
        # the paper form's training step: second stage levels, its batch of four views
        dict(name="paper_step", kind="paper", T=50_000, Rmin=2, Rmax=5, sizes=_text([(800, 800)] * 4),
             loss="l1_ssim", fused=True),
        # the paper form early in training or on a small object: coarse levels, an odd image, separate calls
        dict(name="paper_small_odd", kind="paper", T=3_000, Rmin=1, Rmax=3, sizes="389x517", loss="l2", fused=False),
        # the optimiser over the parameters of a 50,000-triangle soup
        dict(name="optimizer", kind="adam", T=50_000, texel=1024, mlp=1732),
        # the adaptive control between iterations
        dict(name="adapt", kind="adapt", T=50_000, sizes=_text([(800, 800)] * 4), edge_views=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_sizes(rng, lo, hi, most_views, most_pixels):
    sizes, left = [], most_pixels
    for _ in range(_log_int(rng, 1, most_views)):
        s = (_log_int(rng, lo, hi), _log_int(rng, lo, hi))
        if s[0] * s[1] > left:
            break
        sizes.append(s)
        left -= s[0] * s[1]
    return _text(sizes or [(lo, lo)])


def draw(rng):
    kind = rng.choice(["step", "step", "step", "render", "render", "paper", "paper", "adam", "adapt"])
    if kind == "step":
        form = rng.choice(["8-16-4", "16-32-32-4", "16-32-32-4", "32-64-64-4"])
        soup = rng.choice(["ball", "ball", "blobs"])
        api = rng.choice(["calls", "calls", "autograd"])
        return dict(kind="step", form=form, G=rng.choice([4, 8, 8]), T=_log_int(rng, 64, 100_000), soup=soup,
                    sizes=_draw_sizes(rng, 64, 1280, 24, 10_000_000),
                    loss="l2" if api == "autograd" else rng.choice(["l2", "l1_ssim"]), api=api,
                    keep=rng.random() < 0.7)
    if kind == "render":
        soups = sorted({_log_int(rng, 500, 100_000) for _ in range(rng.randint(1, 4))})
        return dict(kind="render", T=",".join(str(t) for t in soups),
                    sizes=_draw_sizes(rng, 120, 1920, 16, 20_000_000))
    if kind == "paper":
        Rmax = rng.choice([3, 4, 5, 5])
        return dict(kind="paper", T=_log_int(rng, 64, 50_000), Rmin=rng.randint(1, Rmax - 1), Rmax=Rmax,
                    sizes=_draw_sizes(rng, 64, 1024, 4, 2_500_000), loss=rng.choice(["l2", "l1_ssim"]),
                    fused=rng.random() < 0.7)
    if kind == "adam":
        return dict(kind="adam", T=_log_int(rng, 64, 50_000), texel=rng.choice([128, 1024, 2048]),
                    mlp=rng.choice([212, 1732, 6532]))
    return dict(kind="adapt", T=_log_int(rng, 500, 50_000), sizes=_draw_sizes(rng, 200, 1024, 4, 2_600_000),
                edge_views=rng.randint(1, 40))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _soup(rng, kind, T):
    if kind == "box":
        return rng.uniform(-1.0, 1.0, (T, 3, 3)).astype(np.float32)
    if kind == "blobs":
        centres = W.uniform_ball(rng, 16)[rng.integers(0, 16, T)] + rng.normal(0.0, 0.15, (T, 3))
    else:
        centres = W.uniform_ball(rng, T)
    return W.equilateral_soup(rng, centres)


def _views(sizes, rng=None):
    """Cameras on the Fibonacci sphere, or (rng) in random directions."""
    n = len(sizes)
    if rng is None:
        eyes = W.fibonacci_sphere(n, 3.0) if n > 1 else np.array([[0.0, 0.0, 3.0]])
    else:
        d = rng.standard_normal((n, 3))
        eyes = 3.0 * d / np.linalg.norm(d, axis=1, keepdims=True)
    return R.Views.from_list([W.View(w, h, i, W.view_proj(eyes[i], w, h)) for i, (w, h) in enumerate(sizes)])


def _inputs(case, seed):
    """The case's inputs as a dict of device tensors and host descriptions."""
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda sd, *shape: torch.randn(*shape, device="cuda", generator=gen) * sd
    host = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    kind = case["kind"]
    if kind == "adam":
        n = [9 * case["T"], case["T"] * case["texel"], case["mlp"]]
        return dict(p=[normal(s, k) for s, k in zip((0.6, 0.1, 0.2), n)], g=[normal(1e-4, k) for k in n],
                    m=[normal(1e-5, k) for k in n],
                    v=[normal(1e-4, k // 3 if i == 0 else k).square() for i, k in enumerate(n)])
    sizes = _sizes(case["sizes"])
    d = dict(seed=0x5EED0000 + seed, views=_views(sizes, rng if kind == "render" else None))
    P = d["views"].pixels
    if kind == "render":
        d["scenes"] = [R.DeviceScene(host(_soup(rng, "ball", int(t))), normal(0.1, int(t), 8, 8, 16),
                                     host(W.glorot_mlp(rng, FORMS["16-32-32-4"])), FORMS["16-32-32-4"])
                       for t in case["T"].split(",")]
        d["which"] = [int(i) for i in rng.permutation(np.arange(len(sizes)) % len(d["scenes"]))]
        return d
    T = case["T"]
    d["verts"] = host(_soup(rng, case.get("soup", "ball"), T))
    if kind == "step":
        dims = FORMS[case["form"]]
        d.update(dims=dims, feats=normal(0.1, T, case["G"], case["G"], dims[0]), mlp=host(W.glorot_mlp(rng, dims)))
    elif kind == "paper":
        d["raw"] = [normal(0.5, T, W.mc_vertices(r), 8) for r in range(case["Rmin"], case["Rmax"])]
        d["mlp"] = host(W.random_pscene(rng, np.zeros((1, 3, 3), np.float32), 0).mlp)
        d["minv"] = R.inv_view_proj(d["views"])
    else:
        d.update(dims=FORMS["16-32-32-4"], feats=normal(0.1, T, 8, 8, 16),
                 mlp=host(W.glorot_mlp(rng, FORMS["16-32-32-4"])))
        d["sample"] = _views([(800, 800)] * case["edge_views"], rng)
        return d
    d["target"] = torch.rand(P, 3, device="cuda", generator=gen)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    d["case"] = case
    if case["kind"] in ("step", "adapt"):
        d["scene"] = R.DeviceScene(d["verts"], d["feats"], d["mlp"], d["dims"])
    if case["kind"] == "adapt":   # the visibility that the training loop's last batch left
        d["vis"] = R.rasterize_fwd(d["scene"], d["views"], R.Opts(seed=d["seed"]))[0]
    if case.get("api") == "autograd":
        d["leaves"] = [d[k].requires_grad_() for k in ("verts", "feats", "mlp")]
    return d


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _loss(d, color):
    if d["case"]["loss"] == "l2":
        return R.loss_l2(color, d["target"])
    return R.loss_l1_ssim(color, d["target"], d["views"])


def _run_step(d):
    opts = R.Opts(seed=d["seed"], reuse_bins=int(d["case"]["keep"]))
    vis, color, _ = R.rasterize_fwd(d["scene"], d["views"], opts)
    loss, gc, gl = _loss(d, color)
    gv, gf, gm = R.rasterize_bwd(d["scene"], d["views"], R.Opts(seed=d["seed"], reuse_bins=1), vis, color, gc, gl)
    return dict(vis=vis, color=color, loss=loss, grad_color=gc, grad_logp=gl, verts=gv, feats=gf, mlp=gm)


def _run_autograd(d):
    for x in d["leaves"]:
        x.grad = None
    color, logp, vis = R.rasterize(*d["leaves"], d["dims"], d["views"], R.Opts(seed=d["seed"]))
    per_pixel = (color - d["target"]).square().sum(1) / (3 * color.shape[0])
    loss = per_pixel.sum()
    (loss + (per_pixel.detach() * logp).sum()).backward()
    gv, gf, gm = (x.grad for x in d["leaves"])
    return dict(vis=vis, color=color.detach(), logp=logp.detach(), loss=loss.detach(), verts=gv, feats=gf, mlp=gm)


def _run_paper(d):
    c = d["case"]
    tex = R.mc_assemble(d["raw"], c["Rmin"], c["Rmax"])
    scene = R.PDeviceScene(d["verts"], tex, d["mlp"], c["Rmax"])
    opts = R.Opts(seed=d["seed"], reuse_bins=1)
    vis, color, _ = R.pforward(scene, d["views"], opts, minv=d["minv"])
    loss, gc, gl = _loss(d, color)
    if c["fused"]:
        gv, graw, gm = R.pbackward_levels(scene, d["views"], opts, vis, color, gc, c["Rmin"], len(d["raw"]), gl,
                                          minv=d["minv"])
    else:
        gv, gt, gm = R.pbackward(scene, d["views"], opts, vis, color, gc, gl, minv=d["minv"])
        graw = R.mc_assemble_bwd(tex, gt, c["Rmin"], len(d["raw"]), c["Rmax"])
    return dict(vis=vis, color=color, loss=loss, grad_color=gc, grad_logp=gl, verts=gv, raw=graw, mlp=gm)


def _run_adapt(d):
    T = d["scene"].T
    counts = R.coverage_count(d["vis"], T)
    rel = R.edge_lengths(d["scene"].verts, d["sample"])
    act, off, n = R.adaptive_plan(counts, rel, target=T, prune_zero=True, fill=True)
    new = R.adaptive_apply(d["scene"], act, off, n)
    return dict(counts=counts, rel=rel, actions=act, verts=new.verts, feats=new.feats)


def run(state):
    d = state
    kind = d["case"]["kind"]
    if kind == "step":
        return _run_autograd(d) if d["case"]["api"] == "autograd" else _run_step(d)
    if kind == "render":
        return R.render([d["scenes"][i] for i in d["which"]], d["views"], R.Opts(mode=1))
    if kind == "paper":
        return _run_paper(d)
    if kind == "adam":
        for i, (lr, vec) in enumerate(((1e-3, 3), (5e-2, 1), (1e-2, 1))):
            R.adam_step(d["p"][i], d["g"][i], d["m"][i], d["v"][i], lr, 10, vec=vec)
        return dict(p=d["p"], m=d["m"], v=d["v"])
    return _run_adapt(d)


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

def _decodes(T, soup, pixels):
    """(fragments up to and with each pixel's winner, winners), expected: T equilateral triangles of
    mean squared side exp(-5.5) at random orientations over the unit disc, which fills 0.294 of a
    square view; a pixel's fragments are Poisson and each passes with probability 1/2."""
    depth = 8.0 if soup == "box" else T * (math.sqrt(3) / 8 * math.exp(-5.5)) / math.pi
    inside = pixels * (1.0 if soup == "box" else 0.294)
    won = inside * (1.0 - math.exp(-0.5 * depth))
    return 2.0 * won, won


def work(case):
    kind, T = case["kind"], case["T"]
    if kind == "adam":
        n = T * case["texel"] + case["mlp"]
        return {"bytes": 28.0 * n + 6 * 4 * 9 * T, "flops": 12.0 * (n + 9 * T)}
    sizes = _sizes(case["sizes"])
    P = float(sum(w * h for w, h in sizes))
    if kind == "render":
        soups = [int(t) for t in T.split(",")]
        flops = sum(2 * 1664 * _decodes(soups[i % len(soups)], "ball", w * min(h, w))[0]
                    for i, (w, h) in enumerate(sizes))
        return {"bytes": sum(soups) * 4132.0 + 12 * P, "flops": flops}
    if kind == "adapt":
        return {"bytes": 8 * P + 48.0 * T + 2 * 4132.0 * T, "flops": 60.0 * T * case["edge_views"]}
    image = P * (8 + 12 + 12 + 12 + 4)   # vis, colour, target, its gradient, score weights
    if kind == "paper":
        levels = sum(W.mc_vertices(r) for r in range(case["Rmin"], case["Rmax"]))
        E, won = _decodes(T, "ball", P)
        return {"bytes": image + T * (72.0 + 2 * 32 * levels + 32 * W.mc_vertices(case["Rmax"])),
                "flops": 8 * 560 * won + 40 * E}
    dims = FORMS[case["form"]]
    mac = sum(a * b for a, b in zip(dims, dims[1:]))
    E, won = _decodes(T, case.get("soup", "ball"), P)
    return {"bytes": image + T * (72.0 + 8 * case["G"] ** 2 * dims[0]), "flops": 8.0 * mac * E + 2.0 * mac * won}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
# Which fragments there are and how they are ordered is decided on float32 positions by definition
# (screen positions are float32 values rounded to 1/256 pixel, a depth is a float32 key), so these
# are formed in float32; every value is float64.

def _fma32(a, b, c):
    return (a.double() * b.double() + c.double()).float()


def _philox_u(seed, pixel, tri, view_id, step):
    """24-bit uniforms of Philox4x32-10 with counter (pixel, tri, view, step), in float64."""
    M32 = 0xFFFFFFFF
    c = [pixel, tri, torch.full_like(pixel, view_id), torch.full_like(pixel, step)]
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & M32) ^ c[1] ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c[3] ^ k1, p0 & M32]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return (c[0] >> 8).double() * 2.0 ** -24


class _View64:
    """One view's fragments: triangle, pixel, key and (through position()) barycentrics."""

    def __init__(self, verts, M, width, height, near=0.1):
        self.W, self.H, self.M = width, height, M.double()
        hw, hh = torch.tensor(0.5 * width, device="cuda"), torch.tensor(0.5 * height, device="cuda")
        c = [_fma32(M[j, 2], verts[..., 2], _fma32(M[j, 1], verts[..., 1], _fma32(M[j, 0], verts[..., 0], M[j, 3])))
             for j in range(4)]
        front = (c[3] >= near).all(1)
        iw = (1.0 / torch.where(c[3] >= near, c[3], torch.ones_like(c[3])).double()).float()
        sx, sy = _fma32(c[0] * iw, hw, hw), _fma32(-(c[1] * iw), hh, hh)
        z = _fma32(c[2] * iw, torch.full_like(hw, 0.5), torch.full_like(hw, 0.5))
        X, Y = torch.round(sx.double() * 256).long(), torch.round(sy.double() * 256).long()
        A = self._edge(X[:, 0], Y[:, 0], X[:, 1], Y[:, 1], X[:, 2], Y[:, 2])
        lo = lambda q, n: ((q.amin(1) + 127) // 256).clamp(0, n)
        hi = lambda q, n: torch.div(q.amax(1) - 128, 256, rounding_mode="floor").clamp(-1, n - 1)
        x0, x1, y0, y1 = lo(X, width), hi(X, width), lo(Y, height), hi(Y, height)
        bw, bh = (x1 - x0 + 1).clamp(min=0), (y1 - y0 + 1).clamp(min=0)
        n = torch.where(front & (A != 0), bw * bh, torch.zeros_like(bw))
        self.X, self.Y, self.A = X, Y, A
        found = []
        ends = torch.cumsum(n, 0).cpu().numpy()
        at = 0
        while at < len(ends):   # triangles in groups of about 2^23 candidate pixels
            to = max(at + 1, int(np.searchsorted(ends, (ends[at - 1] if at else 0) + (1 << 23), "right")))
            t = torch.repeat_interleave(torch.arange(at, to, device="cuda"), n[at:to])
            first = torch.cumsum(n[at:to], 0) - n[at:to]
            k = torch.arange(len(t), device="cuda") - first[t - at]
            px, py = x0[t] + k % bw[t].clamp(min=1), y0[t] + k // bw[t].clamp(min=1)
            s = torch.sign(A[t])
            inside = torch.ones_like(t, dtype=torch.bool)
            E = []
            for i in range(3):
                a, b = (i + 1) % 3, (i + 2) % 3
                e = s * self._edge(X[t, a], Y[t, a], X[t, b], Y[t, b], 256 * px + 128, 256 * py + 128)
                dx, dy = s * (X[t, b] - X[t, a]), s * (Y[t, b] - Y[t, a])
                inside &= (e > 0) | ((e == 0) & ((dy < 0) | ((dy == 0) & (dx > 0))))
                E.append(e)
            t, px, py = t[inside], px[inside], py[inside]
            ra = (1.0 / A[t].abs().float().double()).float()
            beta = [e[inside].float() * ra for e in E]
            depth = _fma32(beta[2], z[t, 2], _fma32(beta[1], z[t, 1], beta[0] * z[t, 0])).clamp(0.0, 1.0) + 0.0
            found.append((t, py * width + px, (depth.view(torch.int32).long() << 32) | t))
            at = to
        self.tri, self.pix, self.key = (torch.cat(f) for f in zip(*found))

    @staticmethod
    def _edge(ax, ay, bx, by, px, py):
        return (bx - ax) * (py - ay) - (by - ay) * (px - ax)

    def position(self, verts, tri, pix):
        """Screen-linear barycentrics, perspective-correct (b1, b2) and screen positions of float64
        vertices [T,3,3]; values at the snapped positions, slopes of the projection itself."""
        v = verts[tri]
        c = [self.M[j, 3] + sum(self.M[j, k] * v[..., k] for k in range(3)) for j in (0, 1, 3)]
        iw = 1.0 / c[2]
        sx, sy = 0.5 * self.W * (c[0] * iw + 1.0), 0.5 * self.H * (1.0 - c[1] * iw)
        sx = self.X[tri].double() / 256 + (sx - sx.detach())
        sy = self.Y[tri].double() / 256 + (sy - sy.detach())
        x, y = (pix % self.W).double() + 0.5, torch.div(pix, self.W, rounding_mode="floor").double() + 0.5
        e = [self._edge(sx[:, (i + 1) % 3], sy[:, (i + 1) % 3], sx[:, (i + 2) % 3], sy[:, (i + 2) % 3], x, y)
             for i in range(3)]
        beta = torch.stack(e, 1) / (e[0] + e[1] + e[2])[:, None]
        t = beta * iw
        b = t[:, 1:] / t.sum(1, keepdim=True)
        return beta, b[:, 0], b[:, 1], sx, sy


def _chunks(n, size=1 << 19):
    return [slice(i, min(n, i + size)) for i in range(0, n, size)]


def _mlp(p, dims, x):
    at = 0
    for l, (i, o) in enumerate(zip(dims, dims[1:])):
        x = x @ p[at:at + i * o].view(o, i).T + p[at + i * o:at + i * o + o]
        at += i * o + o
        x = torch.relu(x) if l + 2 < len(dims) else x
    return x


class _Grid64:
    """The workloads' texture: a bilinear G x G grid of features and the MLP."""

    def __init__(self, feats, mlp, dims):
        self.G, self.dims, self.mlp = feats.shape[1], dims, mlp
        self.rows = feats.reshape(-1, feats.shape[3])

    def logits(self, tri, b1, b2):
        G = self.G
        gx, gy = b1 * (G - 1), b2 * (G - 1)
        ix, iy = gx.detach().floor().long().clamp(0, G - 2), gy.detach().floor().long().clamp(0, G - 2)
        fx, fy = (gx - ix)[:, None], (gy - iy)[:, None]
        at = (tri * G + iy) * G + ix
        T = lambda k: self.rows.index_select(0, at + k)
        x = (1 - fx) * (1 - fy) * T(0) + fx * (1 - fy) * T(1) + (1 - fx) * fy * T(G) + fx * fy * T(G + 1)
        return _mlp(self.mlp, self.dims, x)

    def opacity(self, tri, b1, b2):
        """(alpha, log alpha, log(1 - alpha))"""
        o = self.logits(tri, b1, b2)[:, 3]
        return torch.sigmoid(o), torch.nn.functional.logsigmoid(o), torch.nn.functional.logsigmoid(-o)

    def colour(self, view, tri, b1, b2, pix):
        return torch.sigmoid(self.logits(tri, b1, b2)[:, :3])


def _mc_rows(n, b1, b2):
    """The micro-triangle of (b1, b2) on the grid with n segments an edge: vertex indices and weights [N,3]."""
    u, v = b1 * n, b2 * n
    i = u.detach().floor().long().clamp(0, n - 1)
    j = torch.minimum(v.detach().floor().long().clamp(min=0), n - 1 - i)
    fu, fv = u - i, v - j
    inv = ((fu + fv) > 1) & (i + j <= n - 2)
    index = lambda i, j: j * (n + 1) - j * (j - 1) // 2 + i
    idx = torch.stack([torch.where(inv, index(i + 1, j + 1), index(i, j)), index(i + 1, j), index(i, j + 1)], 1)
    w = torch.stack([torch.where(inv, fu + fv - 1, 1 - fu - fv), torch.where(inv, 1 - fv, fu),
                     torch.where(inv, 1 - fu, fv)], 1)
    return idx, w


def _mc_assemble64(raw, Rmin, Rmax):
    n = 1 << Rmax
    at = torch.tensor([(i, j) for j in range(n + 1) for i in range(n + 1 - j)], device="cuda").double() / n
    z = 0
    for l, r in enumerate(raw):
        idx, w = _mc_rows(1 << (Rmin + l), at[:, 0], at[:, 1])
        z = z + sum(r.index_select(1, idx[:, k]) * w[None, :, k, None] for k in range(3))
    return torch.sigmoid(z)


class _MeshColour64:
    """The paper form's texture [T,V(R),8] and its deferred MLP."""

    def __init__(self, tex, mlp, R_, minv, size):
        self.n, self.V, self.rows, self.mlp = 1 << R_, tex.shape[1], tex.reshape(-1, 8), mlp
        self.minv, self.size = minv, size

    def _at(self, tri, b1, b2):
        idx, w = _mc_rows(self.n, b1, b2)
        idx = idx + (tri * self.V)[:, None]
        return sum(self.rows.index_select(0, idx[:, k]) * w[:, k, None] for k in range(3))

    def opacity(self, tri, b1, b2):
        a = self._at(tri, b1, b2)[:, 7]
        return a, a.log(), torch.log1p(-a)

    def colour(self, view, tri, b1, b2, pix):
        f = self._at(tri, b1, b2)
        Mi = self.minv[view]
        Wd, H = self.size[view]
        x, y = (pix % Wd).double(), torch.div(pix, Wd, rounding_mode="floor").double()
        one = torch.ones_like(x)
        ends = []
        for nz in (-1.0, 1.0):
            p = torch.stack([(2 * x + 1) / Wd - 1, 1 - (2 * y + 1) / H, nz * one, one], 1) @ Mi.T
            ends.append(p[:, :3] / p[:, 3:])
        d = ends[1] - ends[0]
        x, y, z = (d / d.norm(dim=1, keepdim=True)).unbind(1)
        c = [math.sqrt(k / math.pi) for k in (0.25, 0.75, 3.75, 0.3125, 0.9375)]
        sh = torch.stack([c[0] * one, c[1] * y, c[1] * z, c[1] * x, c[2] * x * y, c[2] * y * z,
                          c[3] * (2 * z * z - x * x - y * y), c[2] * x * z, c[4] * (x * x - y * y)], 1)
        m = torch.sigmoid(_mlp(self.mlp, W.PF_MLP_DIMS, torch.cat([f[:, :7], sh], 1)))
        A = f[:, 3:4]
        return A * f[:, :3] + (1 - A) * m


def _forward64(geo, view, view_id, tex, verts, seed, mode):
    """Winners of one view: (colour [P,3], key [P], log p [P], listed fragments, their is-winner)."""
    n = geo.W * geo.H
    passed, lp, lf = [], [], []
    with torch.no_grad():
        for c in _chunks(len(geo.tri)):
            tri, pix = geo.tri[c], geo.pix[c]
            _, b1, b2, _, _ = geo.position(verts, tri, pix)
            alpha, logp, logf = tex.opacity(tri, b1, b2)
            passed.append(_philox_u(seed, pix, tri, view_id, 0) < alpha if mode == 0 else alpha > 0.5)
            lp.append(logp)
            lf.append(logf)
        passed = torch.cat(passed) if passed else torch.zeros(0, dtype=torch.bool, device="cuda")
        key = torch.full((n,), BG_KEY, device="cuda")
        key = key.scatter_reduce(0, geo.pix[passed], geo.key[passed], "amin")
        need = geo.key <= key[geo.pix]
        won = geo.key[need] == key[geo.pix[need]]
        tri, pix = geo.tri[need], geo.pix[need]
        color = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
        for c in _chunks(int(won.sum())):
            t, p = tri[won][c], pix[won][c]
            _, b1, b2, _, _ = geo.position(verts, t, p)
            color[p] = tex.colour(view, t, b1, b2, p)
        logp = torch.zeros(n, dtype=torch.float64, device="cuda")
        if len(tri) and mode == 0:
            logp.index_add_(0, pix, torch.where(won, torch.cat(lp)[need], torch.cat(lf)[need]))
    return color, key, logp, tri, pix, won


def _edge64(key, color, gc, width, height):
    """Per pixel the (x, y) weights of the adjacent pairs in which it is the occluder."""
    k, C, g = key.view(height, width), color.view(height, width, 3), gc.view(height, width, 3)
    out = torch.zeros(height, width, 2, dtype=torch.float64, device="cuda")
    for dim, comp in ((1, 0), (0, 1)):
        n = k.shape[dim]
        ka, kb = k.narrow(dim, 0, n - 1), k.narrow(dim, 1, n - 1)
        w = (0.5 * (g.narrow(dim, 0, n - 1) + g.narrow(dim, 1, n - 1))
             * (C.narrow(dim, 0, n - 1) - C.narrow(dim, 1, n - 1))).sum(2)
        w = torch.where((ka == BG_KEY) & (kb == BG_KEY), torch.zeros_like(w), w)
        out.narrow(dim, 0, n - 1)[..., comp] += torch.where(ka < kb, w, torch.zeros_like(w))
        out.narrow(dim, 1, n - 1)[..., comp] += torch.where(ka < kb, torch.zeros_like(w), w)
    return out.view(-1, 2)


def _backward64(geo, view, tex, verts, frags, gc, gl, edge):
    """Adds one view's gradients to the leaves: the colour path with the draws fixed, the score term
    (which moves no vertex) and the edge term."""
    color, key, _, tri, pix, won = frags
    for c in _chunks(len(tri)):
        t, p, w = tri[c], pix[c], won[c]
        with torch.no_grad():
            _, b1, b2, _, _ = geo.position(verts, t, p)
        _, logp, logf = tex.opacity(t, b1, b2)
        total = (gl[p] * torch.where(w, logp, logf)).sum()
        t, p = t[w], p[w]
        beta, b1, b2, sx, sy = geo.position(verts, t, p)
        total = total + (gc[p] * tex.colour(view, t, b1, b2, p)).sum()
        e = edge[p]
        total = total + (beta.detach() * (e[:, :1] * sx + e[:, 1:] * sy)).sum()
        total.backward()


def _ssim64(x, y):
    g = torch.exp(-torch.arange(-5.0, 6.0, dtype=torch.float64, device="cuda") ** 2 / 4.5)
    g = g / g.sum()

    def blur(z):
        for dim in (0, 1):
            pad = torch.nn.functional.pad(z, (0, 0) + ((5, 5) if dim else (0, 0)) + ((0, 0) if dim else (5, 5)))
            z = sum(g[k] * pad.narrow(dim, k, z.shape[dim]) for k in range(11))
        return z

    mx, my = blur(x), blur(y)
    sxx, syy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    c1, c2 = 1e-4, 9e-4
    return ((2 * mx * my + c1) * (2 * sxy + c2)) / ((mx * mx + my * my + c1) * (sxx + syy + c2))


def _loss64(case, sizes, color, target):
    """(loss, its colour gradient, the per-pixel shares of the loss) over all views."""
    n = color.numel()
    if case["loss"] == "l2":
        d = color - target
        share = d.square().sum(1) / n
        return share.sum(), 2 * d / n, share
    lam, at, grads, shares = 0.8, 0, [], []
    for w, h in sizes:
        x = color[at:at + w * h].view(h, w, 3).requires_grad_()
        y = target[at:at + w * h].view(h, w, 3)
        at += w * h
        share = (lam * (x - y).abs() + (1 - lam) * (1 - _ssim64(x, y))).sum(2) / n
        grads.append(torch.autograd.grad(share.sum(), x)[0].reshape(-1, 3))
        shares.append(share.detach().reshape(-1))
    share = torch.cat(shares)
    return share.sum(), torch.cat(grads), share


def _exact_step(case, d):
    sizes = _sizes(case["sizes"])
    verts = d["verts"].double().requires_grad_()
    mlp = d["mlp"].double().requires_grad_()
    if case["kind"] == "paper":
        raw = [r.double().requires_grad_() for r in d["raw"]]
        assembled = _mc_assemble64(raw, case["Rmin"], case["Rmax"])
        leaf = assembled.detach().requires_grad_()
        tex = _MeshColour64(leaf, mlp, case["Rmax"], torch.from_numpy(d["minv"]).cuda().double(), sizes)
    else:
        feats = d["feats"].double().requires_grad_()
        tex = _Grid64(feats, mlp, d["dims"])
    M = torch.from_numpy(d["views"].view_proj).cuda()
    geos = [_View64(d["verts"], M[i], w, h) for i, (w, h) in enumerate(sizes)]
    fwd = [_forward64(geo, i, i, tex, verts, d["seed"], 0) for i, geo in enumerate(geos)]
    color = torch.cat([f[0] for f in fwd])
    loss, gc, gl = _loss64(case, sizes, color.clone(), d["target"].double())
    at = 0
    for i, (geo, f) in enumerate(zip(geos, fwd)):
        s = slice(at, at + geo.W * geo.H)
        at = s.stop
        _backward64(geo, i, tex, verts, f, gc[s], gl[s], _edge64(f[1], f[0], gc[s], geo.W, geo.H))
    zero = lambda x: torch.zeros_like(x) if x.grad is None else x.grad
    if case["kind"] == "paper":
        assembled.backward(zero(leaf))
    if case.get("api") == "autograd":
        return dict(vis=None, color=color, logp=torch.cat([f[2] for f in fwd]), loss=loss, verts=zero(verts),
                    feats=zero(feats), mlp=zero(mlp))
    out = dict(vis=None, color=color, loss=loss.reshape(1), grad_color=gc, grad_logp=gl, verts=zero(verts))
    out.update(dict(raw=[zero(r) for r in raw]) if case["kind"] == "paper" else dict(feats=zero(feats)))
    return dict(out, mlp=zero(mlp))


def _exact_render(case, d):
    out = []
    M = torch.from_numpy(d["views"].view_proj).cuda()
    for i, (w, h) in enumerate(_sizes(case["sizes"])):
        s = d["scenes"][d["which"][i]]
        tex = _Grid64(s.feats.double(), s.mlp.double(), s.dims)
        out.append(_forward64(_View64(s.verts, M[i], w, h), i, i, tex, s.verts.double(), 0, 1)[0].view(h, w, 3))
    return out


def _exact_adam(d):
    p, m, v = [], [], []
    for i, (lr, vec) in enumerate(((1e-3, 3), (5e-2, 1), (1e-2, 1))):
        g = d["g"][i].double()
        m.append(0.9 * d["m"][i].double() + 0.1 * g)
        v.append(0.999 * d["v"][i].double() + 0.001 * g.view(-1, vec).square().sum(1))
        scale = (v[i] / (1 - 0.999 ** 10)).sqrt() + 1e-8
        p.append(d["p"][i].double() - lr * m[i] / (1 - 0.9 ** 10) / scale.repeat_interleave(vec))
    return dict(p=p, m=m, v=v)


def _exact_adapt(case, d):
    """The edge lengths; the rebuilt soup follows a plan made from counts, and has no value here."""
    v = torch.cat([d["verts"].double(), torch.ones_like(d["verts"][..., :1]).double()], 2)
    best = torch.zeros(case["T"], 3, dtype=torch.float64, device="cuda")
    for M in d["sample"].view_proj:
        c = v @ torch.from_numpy(M).cuda().double().T
        s = torch.stack([400 * (c[..., 0] / c[..., 3] + 1), 400 * (1 - c[..., 1] / c[..., 3])], 2)
        seen = (c[..., 3] >= float(np.float32(0.1))).all(1) & (s.amax(1) >= 0).all(1) & (s.amin(1) <= 800).all(1)
        best = torch.maximum(best, (s.roll(-1, 1) - s).norm(dim=2) / 800 * seen[:, None])
    return dict(counts=None, rel=best, actions=None, verts=None, feats=None)


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "adam":
        return _exact_adam(d)
    if kind == "adapt":
        return _exact_adapt(case, d)
    if kind == "render":
        return _exact_render(case, d)
    return _exact_step(case, d)
