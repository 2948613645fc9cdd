"""The work that users of the denoiser have it do, as measurable cases.

Whole frames through the public objects (one stream, a batch of streams, the
two-channel pipeline, the learned variant), one training step of the
network, and single calls of the library, from the smallest frame to the
largest, in both storage types, 2D and separable, with the options that are
used together.  Inputs are a procedural scene (a ground plane, six spheres, a
sky without surface) seen by a moving camera: the G-buffers of two
consecutive frames, backward motion, one-sample noisy radiance with
fireflies, and the history a running stream holds.

exact() evaluates the same filter in float64 with plain torch, rounding to
the storage type where the filter stores.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2312_06827_amd import learn, lib
from paper_2312_06827_amd.pipeline import (MOTION, BatchDenoiser, ChannelDenoiser, Denoiser,
                                           FilterConfig, FrameInputs)

DEV = "cuda"
D = torch.float64
LUMA = (0.2126, 0.7152, 0.0722)
H5 = (1 / 16, 4 / 16, 6 / 16, 4 / 16, 1 / 16)
G3 = (0.25, 0.5, 0.25)


# ---- the cases ----------------------------------------------------------------

def listed():
    return [
        # the smallest use: a 256x256 preview with a camera at rest (launches
        # and latency count)
        dict(name="frame_small_static", kind="frame", w=256, h=256, half=False, static=True,
             plain=True, separable=False, levels=5),
        # the ordinary use: one 1080p stream, moving camera, clamp, tone map, ids
        dict(name="frame_hd", kind="frame", w=1920, h=1080, half=False, static=False, plain=False,
             separable=False, levels=5),
        # the same with the separable levels
        dict(name="frame_hd_separable", kind="frame", w=1920, h=1080, half=False, static=False,
             plain=False, separable=True, levels=5),
        # the largest frame, in the half storage type
        dict(name="frame_uhd_half", kind="frame", w=3840, h=2160, half=True, static=False,
             plain=False, separable=False, levels=5),
        # an odd window size with history clipping and the blur adapted to
        # roughness (control bytes made every frame)
        dict(name="frame_odd_adaptive_clip", kind="adaptive", w=1365, h=767, half=False,
             separable=False, levels=5),
        # the network inside the temporal step, at its four levels
        dict(name="frame_hd_learned", kind="learned", w=1920, h=1080, half=False, levels=4),
        # shadow and specular channels, adaptive blur, temporal gradient, composition
        dict(name="channels_hd", kind="channels", w=1920, h=1080, half=False),
        # a server's twelve viewers of uneven size in one plan
        dict(name="batch_uneven_half", kind="batch", streams=12, wmin=640, wmax=2560, hmin=360,
             hmax=1440, sizes=4, half=True),
        # one step of training at the trainer's frame size: chain, loss
        # gradients, network backward, Adam
        dict(name="train_step", kind="train", w=320, h=180),
        # the network alone, features to parameter gradient, at full frame size
        dict(name="network_hd", kind="network", w=1920, h=1080),
        # a camera cut: every pixel's history is short, so the variance is
        # the spatial estimate everywhere
        dict(name="variance_cut_hd", kind="variance", w=1920, h=1080, half=False, short=1.0),
        # one level by itself with a kappa map on an odd, pitched window
        dict(name="level_odd_step8", kind="level", w=1283, h=721, pitch=1344, half=False, step=8,
             separable=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo=180, hi=2560):
    """A width over the whole range and a height of a usual aspect."""
    w = _log(rng, lo, hi)
    return w, max(64, int(w / rng.uniform(1.25, 2.4)))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "adaptive", "learned", "channels", "batch",
                       "train", "network", "variance", "level", "level"])
    # the two channels and the network alone cost twice a frame and more
    w, h = _size(rng, hi=1600 if kind in ("channels", "network") else 2560)
    half = rng.random() < 0.4
    if kind == "frame":
        return dict(kind=kind, w=w, h=h, half=half, static=rng.random() < 0.2,
                    plain=rng.random() < 0.2, separable=rng.random() < 0.5,
                    levels=rng.choice([3, 4, 5, 5]))
    if kind == "adaptive":
        return dict(kind=kind, w=w, h=h, half=half, separable=rng.random() < 0.3,
                    levels=rng.choice([4, 5]))
    if kind == "learned":
        return dict(kind=kind, w=w, h=h, half=half, levels=rng.choice([3, 4, 5]))
    if kind == "channels":
        return dict(kind=kind, w=w, h=h, half=half)
    if kind == "batch":
        big = rng.random() < 0.5
        return dict(kind=kind, streams=rng.randint(2, 6 if big else 12), wmin=320 if not big else 640,
                    wmax=640 if not big else 2560, hmin=180 if not big else 360,
                    hmax=360 if not big else 1440, sizes=rng.randrange(1 << 20),
                    half=half or big)
    if kind == "train":
        w, h = _size(rng, 160, 960)
        return dict(kind=kind, w=w, h=h)
    if kind == "network":
        return dict(kind=kind, w=w, h=h)
    if kind == "variance":
        return dict(kind=kind, w=w, h=h, half=half, short=rng.choice([0.02, 0.2, 1.0]))
    return dict(kind=kind, w=w, h=h, pitch=w + rng.choice([0, 0, 1, 61]), half=half,
                step=rng.choice([1, 2, 4, 8, 16]), separable=rng.random() < 0.4)


# ---- inputs -------------------------------------------------------------------

class Scene:
    """Two consecutive frames of the procedural scene, on the GPU."""

    FAR = 45.0  # beyond it the ground has no surface: sky

    def __init__(self, w, h, seed, static=False):
        self.w, self.h, self.static = w, h, static
        r = random.Random(seed)
        self.gen = torch.Generator(device=DEV).manual_seed(seed)
        self.radius = [r.uniform(0.5, 2.0) for _ in range(6)]
        self.center = [[r.uniform(0.0, 10.0) for _ in range(3)] for _ in range(6)]
        self.albedo = torch.tensor([[r.uniform(0.2, 0.9) for _ in range(3)] for _ in range(7)],
                                   dtype=D, device=DEV)
        bands = [0.0, 0.03, 0.1, 0.35, 0.6]
        r.shuffle(bands)
        self.rough = torch.tensor([0.3] + bands + [r.choice(bands)], dtype=torch.float32,
                                  device=DEV)
        self.f = (h / 2.0) / math.tan(math.radians(30.0))
        self.light = torch.tensor([1.0, 2.0, 0.5], dtype=D, device=DEV) / math.sqrt(5.25)
        self.frame = r.randint(1, 40)
        right, up, _ = self._basis(0.0)
        self.vel = []
        for i in range(6):
            a = r.uniform(0, 2 * math.pi)
            s = 0.0 if static or i >= 3 else 5.0 * 12.0 / self.f
            self.vel.append([s * (math.cos(a) * right[k] + math.sin(a) * up[k]) for k in range(3)])

    @staticmethod
    def _basis(yaw):
        fx, fy, fz = 0.0, -9.0, 13.0
        n = math.sqrt(fx * fx + fy * fy + fz * fz)
        fx, fy, fz = fx / n, fy / n, fz / n
        c, s = math.cos(yaw), math.sin(yaw)
        fwd = (c * fx + s * fz, fy, -s * fx + c * fz)
        m = math.hypot(fwd[0], fwd[2])
        right = (fwd[2] / m, 0.0, -fwd[0] / m)
        up = (fwd[1] * right[2] - fwd[2] * right[1], fwd[2] * right[0] - fwd[0] * right[2],
              fwd[0] * right[1] - fwd[1] * right[0])
        return right, up, fwd

    def _camera(self, k):
        if self.static:
            k = 0
        right, up, fwd = self._basis(math.radians(0.1 * k))
        step = 0.0 if self.static else 2.0 * math.sqrt(250.0) / self.f * k
        pos = [5.0 + step * right[0], 9.0, -7.0 + step * right[2]]
        t = lambda v: torch.tensor(v, dtype=D, device=DEV)
        return t(pos), t(right), t(up), t(fwd)

    def _centers(self, k):
        return [torch.tensor([c[j] + k * v[j] for j in range(3)], dtype=D, device=DEV)
                for c, v in zip(self.center, self.vel)]

    def gbuffer(self, k):
        w, h, f = self.w, self.h, self.f
        pos, right, up, fwd = self._camera(k)
        u = (torch.arange(w, dtype=D, device=DEV) + 0.5 - w / 2.0) / f
        v = -(torch.arange(h, dtype=D, device=DEV) + 0.5 - h / 2.0) / f
        d = fwd[:, None, None] + u[None, None, :] * right[:, None, None] \
            + v[None, :, None] * up[:, None, None]
        inf = torch.full((h, w), math.inf, dtype=D, device=DEV)
        z = torch.where(d[1] < 0, -pos[1] / d[1], inf)
        z = torch.where(z < self.FAR, z, inf)
        obj = torch.zeros((h, w), dtype=torch.int64, device=DEV)
        a = (d * d).sum(0)
        centers = self._centers(k)
        for i, s in enumerate(centers):
            oc = pos - s
            b = 2.0 * (oc[:, None, None] * d).sum(0)
            disc = b * b - 4.0 * a * (float(oc @ oc) - self.radius[i] ** 2)
            t = (-b - disc.clamp_min(0).sqrt()) / (2.0 * a)
            hit = (disc > 0) & (t > 1e-6) & (t < z)
            z = torch.where(hit, t, z)
            obj = torch.where(hit, torch.full_like(obj, i + 1), obj)
        sky = torch.isinf(z)
        x = pos[:, None, None] + torch.where(sky, torch.zeros_like(z), z) * d
        n = torch.zeros((3, h, w), dtype=D, device=DEV)
        n[1] = 1.0
        for i, s in enumerate(centers):
            m = obj == i + 1
            n = torch.where(m, (x - s[:, None, None]) / self.radius[i], n)
        n = n / (n * n).sum(0).sqrt()
        nd = (n * d).sum(0)
        nd = torch.where(nd.abs() < 1e-6, torch.full_like(nd, -1e-6), nd)
        zero = torch.zeros_like(z)
        gx = torch.where(sky, zero, -z * (right[:, None, None] * n).sum(0) / (f * nd))
        gy = torch.where(sky, zero, z * (up[:, None, None] * n).sum(0) / (f * nd))
        return dict(z=torch.where(sky, zero, z), dzdx=gx, dzdy=gy, n=n, obj=obj, x=x, sky=sky)

    def _project(self, x, k, gb):
        pos, right, up, fwd = self._camera(k)
        rel = x - pos[:, None, None]
        zc = (fwd[:, None, None] * rel).sum(0)
        zs = torch.where(gb["sky"], torch.ones_like(zc), zc)
        px = (right[:, None, None] * rel).sum(0) / zs * self.f + self.w / 2.0 - 0.5
        py = -(up[:, None, None] * rel).sum(0) / zs * self.f + self.h / 2.0 - 0.5
        mv = torch.stack([px - torch.arange(self.w, dtype=D, device=DEV)[None, :],
                          py - torch.arange(self.h, dtype=D, device=DEV)[:, None]])
        return torch.where(gb["sky"] | (zc < 0.1), torch.zeros_like(mv), mv), zc

    def motion(self, gb, k, to):
        """Where each surface point of frame k is seen in frame `to`."""
        x = gb["x"]
        if self.static:
            return torch.zeros((2, self.h, self.w), dtype=D, device=DEV), gb["z"]
        for i in range(6):
            m = gb["obj"] == i + 1
            v = torch.tensor(self.vel[i], dtype=D, device=DEV) * (to - k)
            x = torch.where(m, x + v[:, None, None], x)
        return self._project(x, to, gb)

    def shade(self, gb):
        lit = (self.light[:, None, None] * gb["n"]).sum(0).clamp_min(0.0)
        c = self.albedo[gb["obj"]].permute(2, 0, 1) * lit
        return torch.where(gb["sky"], torch.full_like(c, 0.6), c)

    def rand(self, *shape):
        return torch.rand(shape, dtype=D, device=DEV, generator=self.gen)

    def noisy(self, clean):
        e = -torch.log1p(-self.rand(*clean.shape))
        fire = self.rand(*clean.shape[1:]) < 0.005
        return clean * e * torch.where(fire, 50.0, 1.0) / 1.245


def _inputs(case, seed):
    """(scene, FrameInputs, history, extras) of one running stream."""
    w, h = case["w"], case["h"]
    ft = torch.float16 if case.get("half") else torch.float32
    s = Scene(w, h, seed, case.get("static", False))
    g1, g0 = s.gbuffer(s.frame), s.gbuffer(s.frame - 1)
    q = lambda t: t.to(torch.float32).to(ft).contiguous()
    u8 = lambda t: t.to(torch.uint8).contiguous()
    clean = s.shade(g1)
    mv, _ = s.motion(g1, s.frame, s.frame - 1)
    inp = FrameInputs(
        rgb=q(s.noisy(clean)), g=lib.GBuf(q(g1["z"]), q(g1["dzdx"]), q(g1["dzdy"]), q(g1["n"]),
                                          u8(g1["obj"])),
        mv=q(mv), prev=lib.GBuf(q(g0["z"]), None, None, q(g0["n"]), u8(g0["obj"])),
        albedo=q(s.albedo[g1["obj"]].permute(2, 0, 1)))
    # what a stream holds after a dozen frames: the filtered colour of the
    # last one, its moments, and a short history where the camera just came
    c0 = s.shade(g0)
    if not case.get("plain"):
        c0 = c0 / (1.0 + _luma(c0))
    c0 = c0 * (1.0 + 0.1 * (s.rand(3, h, w) - 0.5))
    m1 = _luma(c0) * (1.0 + 0.2 * (s.rand(h, w) - 0.5))
    m2c = (0.4 * m1) ** 2 * -torch.log1p(-s.rand(h, w))
    n = torch.full((h, w), 12, dtype=torch.uint8, device=DEV)
    n[:, -6:] = (torch.arange(6, device=DEV).flip(0) // 2 + 1).to(torch.uint8)
    n = torch.where(g0["sky"], torch.zeros_like(n), n)
    zero = torch.zeros_like(m1)
    hist = dict(rgb=q(c0), m1=torch.where(g0["sky"], zero, m1).float(),
                m2c=torch.where(g0["sky"], zero, m2c).float(), n=n)
    return s, inp, hist, dict(g1=g1, g0=g0, clean=clean.float().contiguous())


def _config(case):
    if case["kind"] == "adaptive":
        return FilterConfig(clip=True, tonemap=True, use_id=True, levels=case["levels"],
                            separable=case["separable"])
    if case.get("plain"):
        return FilterConfig(levels=case["levels"], separable=case["separable"])
    if case["kind"] in ("batch", "train"):
        return MOTION
    return FilterConfig(clamp=True, tonemap=True, use_id=True, levels=case["levels"],
                        separable=case.get("separable", False))


def _load_history(den, hist):
    for name, t in (("c_hist", hist["rgb"]), ("m1", hist["m1"]), ("m2c", hist["m2c"]),
                    ("n", hist["n"])):
        getattr(den, name)[0].copy_(t)


def _batch_cases(case):
    r = random.Random(case["sizes"])
    return [dict(kind="frame", w=r.randint(case["wmin"], case["wmax"]),
                 h=r.randint(case["hmin"], case["hmax"]), half=case["half"])
            for _ in range(case["streams"])]


def _channels(case, seed):
    """The two channels' samples and the temporal gradient's inputs."""
    s, inp, hist, ex = _inputs(case, seed)
    g1, g0 = ex["g1"], ex["g0"]
    ft = torch.float16 if case["half"] else torch.float32
    q = lambda t: t.to(torch.float32).to(ft).contiguous()

    def visibility(x, k):
        # a penumbra around every sphere's shadow on the other surfaces
        v = torch.ones(x.shape[1:], dtype=D, device=DEV)
        for c, r in zip(s._centers(k), s.radius):
            d = c[:, None, None] - x
            along = (s.light[:, None, None] * d).sum(0)
            off = (d - along * s.light[:, None, None]).pow(2).sum(0).sqrt()
            soft = 0.07 * along.clamp_min(0.5)
            v = v * torch.where(along > 0.2 + r, ((off - r) / soft + 0.5).clamp(0, 1),
                                torch.ones_like(v))
        return v

    u_prev, u_cur = s.rand(case["h"], case["w"]), s.rand(case["h"], case["w"])
    vis0, vis1 = visibility(g0["x"], s.frame - 1), visibility(g1["x"], s.frame)
    three = lambda t: t.to(D).expand(3, -1, -1)
    shadow, shadow0 = q(three(u_cur < vis1)), q(three(u_prev < vis0))
    fmv, fz = s.motion(g0, s.frame - 1, s.frame)
    again = q(three(u_prev < vis0 * (1.0 - 0.2 * (vis0 < 0.7))))
    rough = s.rough[g1["obj"]].contiguous()
    spec_clean = three(0.5 * (1.0 - rough.to(D))) * (0.5 + 0.5 * g1["n"][1])
    h, w = case["h"], case["w"]
    pick = torch.randint(0, 9, ((h + 2) // 3, (w + 2) // 3), generator=s.gen, device=DEV,
                         dtype=torch.uint8)
    # histories: the filtered visibility and the tone-mapped specular light
    sh = {k: v.clone() for k, v in hist.items()}
    v0 = (vis0 * (1.0 + 0.02 * (s.rand(h, w) - 0.5))).clamp(0, 1)
    sh["rgb"] = q(three(v0))
    sh["m1"], sh["m2c"] = v0.float(), (v0 * (1 - v0)).float()
    sp = {k: v.clone() for k, v in hist.items()}
    p0 = spec_clean / (1.0 + _luma(spec_clean))
    sp["rgb"] = q(p0 * (1.0 + 0.1 * (s.rand(3, h, w) - 0.5)))
    sp["m1"] = _luma(p0).float()
    sp["m2c"] = ((0.4 * _luma(p0)) ** 2).float()
    return dict(inp=inp, shadow=shadow, spec=q(s.noisy(spec_clean)), direct=q(ex["clean"]),
                rough=rough, angle=torch.full((h, w), 8.0, device=DEV),
                grad=dict(prev=shadow0, reshade=again, fmv=q(fmv), fz=q(fz), pick=pick),
                hist=[sh, sp])


def _pitched(t, pitch):
    """The same plane (or planes) with a row pitch of `pitch` elements."""
    if pitch == t.shape[-1]:
        return t.contiguous()
    big = torch.zeros((*t.shape[:-1], pitch), dtype=t.dtype, device=t.device)
    v = big[..., :t.shape[-1]]
    v.copy_(t)
    return v


def _level_inputs(case, seed):
    s, inp, hist, _ = _inputs(dict(case, plain=True), seed)
    p = case["pitch"]
    v = torch.where(inp.g.z > 0, hist["m2c"], torch.zeros_like(hist["m2c"]))
    kappa = (0.5 + s.rand(case["h"], case["w"])).float()
    g = inp.g
    return dict(c=_pitched(hist["rgb"], p), v=_pitched(v, p), kappa=_pitched(kappa, p),
                g=lib.GBuf(_pitched(g.z, p), _pitched(g.dzdx, p), _pitched(g.dzdy, p),
                           _pitched(g.n, p)))


def _network_inputs(case, seed):
    s, inp, hist, _ = _inputs(case, seed)
    h, w = case["h"], case["w"]
    return inp, hist, ((s.rand(h, w) - 0.5) * 0.2).float(), ((s.rand(h, w) - 0.5) * 0.1).float()


def _variance_inputs(case, seed):
    s, inp, hist, _ = _inputs(case, seed)
    h, w = case["h"], case["w"]
    # the short pixels come in patches, as disocclusions and cuts do
    r = torch.rand(((h + 15) // 16, (w + 15) // 16), generator=s.gen, device=DEV)
    m = (r < case["short"]).repeat_interleave(16, 0).repeat_interleave(16, 1)[:h, :w]
    n = torch.where(m, torch.randint(1, 4, (h, w), generator=s.gen, device=DEV,
                                     dtype=torch.uint8), torch.full_like(hist["n"], 12))
    live = inp.g.z > 0
    return inp.g, torch.where(live, hist["m1"], 0.0), torch.where(live, hist["m2c"], 0.0), \
        torch.where(live, n, torch.zeros_like(n))


def prepare(case, seed):
    k, h = case["kind"], case.get("h")
    ft = torch.float16 if case.get("half") else torch.float32
    st = dict(kind=k)
    if k in ("frame", "adaptive", "learned"):
        s, inp, hist, _ = _inputs(case, seed)
        den = Denoiser(h, case["w"], _config(case), dtype=ft,
                       mlp=learn.load_weights() if k == "learned" else None)
        _load_history(den, hist)
        st.update(den=den, inp=inp)
        if k == "adaptive":
            inp.blur_ctl = torch.zeros((h, case["w"]), dtype=torch.uint8, device=DEV)
            st.update(rough=s.rough[s.gbuffer(s.frame)["obj"]].contiguous(), rule=lib.BlurRule())
    elif k == "batch":
        cases = _batch_cases(case)
        den = BatchDenoiser([(c["h"], c["w"]) for c in cases], MOTION, dtype=ft)
        ins = []
        for i, (c, d) in enumerate(zip(cases, den.streams)):
            _, inp, hist, _ = _inputs(c, seed + 1000 * i)
            _load_history(d, hist)
            ins.append(inp)
        st.update(den=den, ins=ins)
    elif k == "channels":
        c = _channels(case, seed)
        den = ChannelDenoiser(h, case["w"], dtype=ft)
        for d, hist in zip(den.batch.streams, c["hist"]):
            _load_history(d, hist)
        st.update(den=den, c=c)
    elif k == "train":
        _, inp, hist, ex = _inputs(case, seed)
        mlp = learn.load_weights()
        den = learn.LearnedDenoiser(h, case["w"], mlp, MOTION)
        _load_history(den, hist)
        st.update(den=den, inp=inp, clean=ex["clean"], mlp=mlp)
    elif k == "network":
        inp, hist, da, dk = _network_inputs(case, seed)
        like = torch.empty((h, case["w"]), dtype=torch.float32, device=DEV)
        mlp = learn.load_weights()
        st.update(inp=inp, hist=hist, da=da, dk=dk, mlp=mlp, like=like,
                  feat=lib.feature_rows(h, case["w"]), alpha=torch.empty_like(like),
                  kappa=torch.empty_like(like), work=lib.mlp_workspace(like),
                  grad=torch.empty(lib.SV_MLP_PARAMS, dtype=torch.float32, device=DEV),
                  params=MOTION.temporal())
    elif k == "variance":
        g, m1, m2c, n = _variance_inputs(case, seed)
        var = torch.empty_like(m1)
        st.update(g=g, m1=m1, m2c=m2c, n=n, var=var, work=lib.variance_workspace(var),
                  params=FilterConfig().variance())
    else:
        li = _level_inputs(case, seed)
        p = case["pitch"]
        st.update(li, out=_pitched(torch.zeros_like(li["c"]), p),
                  vout=_pitched(torch.zeros_like(li["v"]), p), step=case["step"],
                  separable=case["separable"], params=FilterConfig().atrous())
    return st


# ---- one pass -----------------------------------------------------------------

def _stream_outputs(den):
    return dict(out=den.out, **den.state())


def run(st):
    k = st["kind"]
    if k in ("frame", "learned"):
        st["den"].frame(st["inp"])
        return _stream_outputs(st["den"])
    if k == "adaptive":
        lib.sv_blur_control(st["rough"], None, st["inp"].blur_ctl, st["rule"])
        st["den"].frame(st["inp"])
        return _stream_outputs(st["den"])
    if k == "batch":
        st["den"].frame(st["ins"])
        return [_stream_outputs(d) for d in st["den"].streams]
    if k == "channels":
        c = st["c"]
        out = st["den"].frame(c["inp"], c["shadow"], c["spec"], c["direct"], c["rough"],
                              c["angle"], c["grad"])
        return dict(out=out, alpha=st["den"].grad_alpha,
                    streams=[_stream_outputs(d) for d in st["den"].batch.streams])
    if k == "train":
        den, mlp = st["den"], st["mlp"]
        out = den.frame(st["inp"], st["inp"].albedo, st["clean"], train=True)
        lib.sv_adam(mlp, den.grad, lr=1e-3)
        return dict(out=out, d_alpha=den.d_alpha, d_kappa=den.d_kappa, grad=den.grad,
                    params=mlp.params, m=mlp.m, v=mlp.v)
    if k == "network":
        inp, hist, mlp = st["inp"], st["hist"], st["mlp"]
        lib.sv_mlp_features(inp.rgb, inp.g, inp.mv, inp.prev, hist["rgb"], hist["m1"],
                            hist["m2c"], hist["n"], inp.albedo, mlp, st["feat"], st["params"])
        lib.sv_mlp_forward(mlp, st["feat"], st["alpha"], st["kappa"], st["like"])
        lib.sv_mlp_backward(mlp, st["feat"], st["da"], st["dk"], st["grad"], st["work"],
                            st["like"], scale=1.0 / st["like"].numel())
        return dict(alpha=st["alpha"], kappa=st["kappa"], grad=st["grad"])
    if k == "variance":
        lib.sv_variance(st["m1"], st["m2c"], st["n"], st["g"], st["var"], st["params"],
                        st["work"])
        return st["var"]
    if st["separable"]:
        lib.sv_atrous_sep(st["c"], st["v"], st["g"], None, st["out"], st["vout"], st["step"],
                          st["params"], kappa=st["kappa"])
    else:
        lib.sv_atrous(st["c"], st["v"], st["g"], st["out"], st["vout"], st["step"], st["params"],
                      kappa=st["kappa"])
    return dict(out=st["out"], var=st["vout"])


# ---- what a pass cannot do without --------------------------------------------

def work(case):
    """Bytes of the inputs read once and the outputs written once; operations
    of the filter's definition (an exponential counted as one)."""
    k = case["kind"]
    if k == "batch":
        ws = [work(dict(c, levels=5)) for c in _batch_cases(case)]
        return {x: sum(v[x] for v in ws) for x in ("bytes", "flops")}
    px = case["w"] * case["h"]
    e = 2 if case.get("half") else 4
    # colour, z, gradients, normal, motion, previous z and normal, history
    # colour; ids, moments and lengths / output, history and state
    frame_b = 18 * e + 2 + 9 + 6 * e + 9
    level_f = 24 * 34 + 120
    sep_f = 8 * 34 + 80
    temporal_f = 300
    net_f = 2 * (14 * 32 + 32 * 32 + 32 * 2)
    if k in ("frame", "adaptive", "learned"):
        lf = sep_f if case.get("separable") else level_f
        b, f = frame_b, temporal_f + case["levels"] * lf
        if k == "adaptive":
            b += 4
        if k == "learned":
            b, f = b + 3 * e, f + net_f
    elif k == "channels":
        b = 2 * frame_b - 10 * e + 3 * e + 3 * e + 8 + (3 + 3 + 2 + 1) * e / 9 + 4
        f = 2 * (temporal_f + 4 * level_f) + 3 * level_f / 9
    elif k == "train":
        b = frame_b + 3 * e + 12 + 8
        f = 2 * temporal_f + 5 * 3 * level_f + 4 * net_f
    elif k == "network":
        b, f = 18 * 4 + 2 + 9 + 12 + 16, temporal_f + 4 * net_f
    elif k == "variance":
        b, f = 6 * e + 9 + 4, case["short"] * 49 * 40 + 4
    else:
        b, f = 9 * e + 8 + 3 * e + 4, sep_f if case["separable"] else level_f
    return dict(bytes=float(px * b), flops=float(px * f))


# ---- the filter in float64 ----------------------------------------------------

def _luma(c):
    return LUMA[0] * c[0] + LUMA[1] * c[1] + LUMA[2] * c[2]


def _sh(t, dx, dy, fill=0.0):
    """t at (x + dx, y + dy); `fill` outside the image."""
    h, w = t.shape[-2:]
    out = torch.full_like(t, fill)
    x0, x1, y0, y1 = max(0, -dx), min(w, w - dx), max(0, -dy), min(h, h - dy)
    if x0 < x1 and y0 < y1:
        out[..., y0:y1, x0:x1] = t[..., y0 + dy:y1 + dy, x0 + dx:x1 + dx]
    return out


def _rounder(half):
    if half:
        return lambda t: t.to(torch.float16).to(D)
    return lambda t: t


def _gb(g):
    z = g.z.to(D)
    live = (g.z > 0) & torch.isfinite(g.z)
    return dict(z=z, live=live, n=g.n.to(D), gx=g.dzdx.to(D), gy=g.dzdy.to(D))


def _xtemporal(inp, hist, cfg, alpha=None, net=None):
    """History accumulation; `net`: (features -> alpha, kappa) of the learned
    step.  Returns a dict of colour, moments, length, clamped history, kappa."""
    f32 = torch.float32
    z, n = inp.g.z.to(f32), inp.g.n.to(f32)
    h, w = z.shape
    live = (z > 0) & torch.isfinite(z)
    c = inp.rgb.to(D)
    if cfg.tonemap:
        c = c / (1.0 + cfg.tm_k * _luma(c))
    lum = _luma(c)
    mv = inp.mv.to(f32)
    fl = torch.floor(mv)
    frac = [(mv[i].to(D) - fl[i].to(D)) for i in range(2)]
    x0 = torch.arange(w, device=DEV)[None, :] + fl[0].long()
    y0 = torch.arange(h, device=DEV)[:, None] + fl[1].long()
    pz, pn = inp.prev.z.to(f32), inp.prev.n.to(f32)
    ids = inp.g.id, inp.prev.id
    hr = hist["rgb"].to(D)
    taps = []
    for t in range(4):
        tx, ty = x0 + (t & 1), y0 + (t >> 1)
        b = (frac[0] if t & 1 else 1.0 - frac[0]) * (frac[1] if t >> 1 else 1.0 - frac[1])
        inside = (tx >= 0) & (tx < w) & (ty >= 0) & (ty < h) & (b > 0)
        i = torch.where(inside, ty * w + tx, torch.zeros_like(tx))
        at = lambda p: p.reshape(*p.shape[:-2], -1)[..., i]
        zt, nt = at(pz), at(pn)
        cos = (nt[2].to(D) * n[2].to(D) + (nt[1].to(D) * n[1].to(D) + (nt[0] * n[0]).to(D))
               .to(f32).to(D)).to(f32)
        ok = inside & (at(hist["n"]) >= 1) & ((zt - z).abs() <= (cfg.tau_z * z)) & \
            (cos >= torch.tensor(cfg.tau_n, dtype=f32)) & live
        if cfg.use_id:
            ok = ok & (at(ids[1]) == ids[0])
        b = torch.where(ok, b, torch.zeros_like(b))
        taps.append((ok, b, at(hr), at(hist["m1"].to(D)), at(hist["m2c"].to(D)),
                     at(hist["n"].long())))
    sw = sum(t[1] for t in taps)
    have = taps[0][0] | taps[1][0] | taps[2][0] | taps[3][0]
    sd = torch.where(have, sw, torch.ones_like(sw))
    hc = sum(t[1] * t[2] for t in taps) / sd
    h1 = sum(t[1] * t[3] for t in taps) / sd
    h2 = sum(t[1] * (t[4] + (t[3] - h1) ** 2) for t in taps) / sd
    nm = torch.stack([torch.where(t[0], t[5], torch.zeros_like(t[5])) for t in taps]).amax(0)
    # the 3x3 box of the current colour
    cnt = sum(_sh(live.to(D), i - 1, j - 1) for i in range(3) for j in range(3)).clamp_min(1)
    cl = torch.where(live, c, torch.zeros_like(c))
    mu = sum(_sh(cl, i - 1, j - 1) for i in range(3) for j in range(3)) / cnt
    var = sum(_sh(live.to(D), i - 1, j - 1) * (_sh(cl, i - 1, j - 1) - mu) ** 2
              for i in range(3) for j in range(3)) / cnt
    half = cfg.gamma * var.sqrt()
    if cfg.clamp:
        hc = torch.minimum(torch.maximum(hc, mu - half), mu + half)
    elif cfg.clip:
        d = hc - mu
        t = torch.where(d.abs() > half, half / d.abs().clamp_min(1e-300),
                        torch.ones_like(d)).amin(0)
        hc = torch.where(t < 1, mu + t * d, hc)
    new = torch.where(have, (nm + 1).clamp_max(cfg.max_hist), torch.ones_like(nm))
    kappa = None
    if net is not None:
        mean = _luma(mu)
        lv = sum(_sh(live.to(D), i - 1, j - 1) * (_sh(_luma(cl), i - 1, j - 1) - mean) ** 2
                 for i in range(3) for j in range(3)) / cnt
        zero = torch.zeros_like(lum)
        mvd = mv.to(D)
        feat = torch.stack([lum, torch.where(have, _luma(hc), zero),
                            torch.where(have, h2.clamp_min(0), zero), lv, new.to(D) / 255.0,
                            inp.g.dzdx.to(D), inp.g.dzdy.to(D), *n.to(D),
                            (mvd[0] ** 2 + mvd[1] ** 2).sqrt(), *inp.albedo.to(D)])
        feat = torch.where(live, feat, torch.zeros_like(feat))
        net = net(feat.reshape(14, -1))
        alpha, kappa = net["alpha"].reshape(h, w), net["kappa"].reshape(h, w)
    inv = 1.0 / new.to(D)
    a = torch.full_like(inv, cfg.alpha) if alpha is None else alpha.to(D)
    ac, am = torch.maximum(a, inv), inv.clamp_min(cfg.alpha_m)
    dl = lum - h1
    out = torch.where(have, hc + ac * (c - hc), c)
    m1 = torch.where(have, h1 + am * dl, lum)
    m2 = torch.where(have, (1 - am) * (h2 + am * dl * dl), torch.zeros_like(lum))
    zero = torch.zeros_like(lum)
    return dict(rgb=torch.where(live, out, c), m1=torch.where(live, m1, zero),
                m2c=torch.where(live, m2, zero),
                n=torch.where(live, new, torch.zeros_like(new)),
                hist=torch.where(have & live, hc, torch.zeros_like(hc)), cur=c, alpha=alpha,
                kappa=kappa, net=net)


def _wn(n, q):
    """Cosine (chord form) of the normals, floored at 0, to the power 128."""
    return (1.0 - 0.5 * ((n - q) ** 2).sum(0)).clamp_min(0.0) ** 128.0


def _xvariance(m1, m2c, n, g):
    s0, s1, s2 = torch.zeros_like(m1), torch.zeros_like(m1), torch.zeros_like(m1)
    live = g["live"].to(D)
    for dy in range(-3, 4):
        for dx in range(-3, 4):
            if dx or dy:
                zq = _sh(g["z"], dx, dy)
                wz = torch.exp(-(g["z"] - zq).abs() /
                               ((g["gx"] * dx + g["gy"] * dy).abs() + 1e-10))
                w = wz * _wn(g["n"], _sh(g["n"], dx, dy)) * _sh(live, dx, dy)
            else:
                w = live
            s0 += w
            s1 += w * _sh(m1, dx, dy)
            s2 += w * _sh(m2c, dx, dy)
    s0 = s0.clamp_min(1e-300)
    mean = s1 / s0
    sp = torch.zeros_like(m1)
    for dy in range(-3, 4):
        for dx in range(-3, 4):
            if dx or dy:
                zq = _sh(g["z"], dx, dy)
                wz = torch.exp(-(g["z"] - zq).abs() /
                               ((g["gx"] * dx + g["gy"] * dy).abs() + 1e-10))
                w = wz * _wn(g["n"], _sh(g["n"], dx, dy)) * _sh(live, dx, dy)
            else:
                w = live
            sp += w * (_sh(m1, dx, dy) - mean) ** 2
    spatial = ((s2 + sp) / s0).clamp_min(0.0)
    v = torch.where(n >= 4, m2c.clamp_min(0.0), spatial)
    return torch.where(g["live"] & (n >= 1), v, torch.zeros_like(v))


def _xprefilter(v, g):
    live = g["live"].to(D)
    s, sw = torch.zeros_like(v), torch.zeros_like(v)
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            k = G3[dx + 1] * G3[dy + 1] * _sh(live, dx, dy)
            s += k * _sh(v, dx, dy)
            sw += k
    return s / sw.clamp_min(1e-300)


def _xpass(c, v, pf, g, kappa, offs, sl=4.0, terms=None):
    """One weighted pass over the taps `offs` = ((dx, dy, H), ...).  With
    `terms` it also sums the derivative by kappa."""
    lum = _luma(c)
    sd = pf.clamp_min(0).sqrt()
    k = 1.0 if kappa is None else kappa
    den = sl * k * sd + 1e-10
    sw = torch.zeros_like(lum)
    sc, sv = torch.zeros_like(c), torch.zeros_like(lum)
    d0, dc = torch.zeros_like(lum), torch.zeros_like(c)
    for dx, dy, hh in offs:
        if dx or dy:
            live = _sh(g["live"].to(D), dx, dy)
            cq = _sh(c, dx, dy)
            w = torch.exp(-(g["z"] - _sh(g["z"], dx, dy)).abs() /
                          ((g["gx"] * dx + g["gy"] * dy).abs() + 1e-10))
            dl = (lum - _luma(cq)).abs()
            w = w * _wn(g["n"], _sh(g["n"], dx, dy)) * torch.exp(-dl / den) * live
            if terms is not None:
                dw = hh * w * dl * sl * sd / (den * den)
                d0 += dw
                dc += dw * cq
            w = hh * w
            sw += w
            sc += w * cq
            sv += w * w * _sh(v, dx, dy)
        else:
            sw += hh
            sc += hh * c
            sv += hh * hh * v
    out, var = sc / sw, sv / (sw * sw)
    if terms is not None:
        terms.append((dc - out * d0) / sw)
    out = torch.where(g["live"], out, c)
    return out, torch.where(g["live"], var, torch.zeros_like(var))


def _taps(step, form):
    if form == "h":
        return [(step * a, 0, H5[a + 2]) for a in range(-2, 3)]
    if form == "v":
        return [(0, step * a, H5[a + 2]) for a in range(-2, 3)]
    return [(step * a, step * b, H5[a + 2] * H5[b + 2]) for b in range(-2, 3)
            for a in range(-2, 3)]


def _xlevel(c, v, g, kappa, step, separable, q, terms=None):
    pf = _xprefilter(v, g)
    if not separable:
        return _xpass(c, v, pf, g, kappa, _taps(step, "2d"), terms=terms)
    hc, _ = _xpass(c, v, pf, g, kappa, _taps(step, "h"))
    return _xpass(q(hc), v, pf, g, kappa, _taps(step, "v"))


def _xchain(t, inp, cfg, half, kappa=None, ctl=None):
    """Variance and levels after the temporal step `t`."""
    q = _rounder(half)
    g = _gb(inp.g)
    c = q(t["rgb"])
    v = _xvariance(t["m1"], t["m2c"], t["n"], g)
    first = None
    for i in range(cfg.levels):
        oc, ov = _xlevel(c, v, g, kappa, 1 << i, cfg.separable, q)
        if ctl is not None:
            sc, s_v = _xlevel(c, v, g, kappa, 2 << i, cfg.separable, q)
            shifted, spent = (ctl & 16) != 0, (ctl & 15) <= i
            oc = torch.where(spent, c, torch.where(shifted, sc, oc))
            ov = torch.where(spent, v, torch.where(shifted, s_v, ov))
        if i == cfg.levels - 1 and cfg.tonemap:
            last = oc / (1.0 - cfg.tm_k * _luma(oc)).clamp_min(2.0 ** -20)
        else:
            last = oc
        c, v = q(oc), ov
        first = c if first is None else first
    return dict(out=q(last), rgb=first, m1=t["m1"], m2c=t["m2c"], n=t["n"])


def _bf(t):
    return t.to(torch.bfloat16).to(D)


def _network(mlp):
    """The network on raw features (14, N), with bfloat16 operands."""
    p = mlp.params.to(D)
    wq = _bf(mlp.params)
    w1, b1 = wq[:448].reshape(32, 14), p[448:480]
    w2, b2 = wq[480:1504].reshape(32, 32), p[1504:1536]
    w3, b3 = wq[1536:1600].reshape(2, 32), p[1600:1602]

    def run_net(f):
        x = _bf((f - mlp.mu.to(D)[:, None]) * mlp.inv_s.to(D)[:, None])
        a1 = w1 @ x + b1[:, None]
        h1 = _bf(a1.clamp_min(0))
        a2 = w2 @ h1 + b2[:, None]
        h2 = _bf(a2.clamp_min(0))
        o = w3 @ h2 + b3[:, None]
        return dict(x=x, a1=a1, h1=h1, a2=a2, h2=h2, o=o,
                    alpha=0.05 + 0.95 * torch.sigmoid(o[0]),
                    kappa=torch.exp2(2.0 * torch.tanh(o[1])), w2=w2, w3=w3)
    return run_net


def _xbackward(net, da, dk):
    s = torch.sigmoid(net["o"][0])
    e = torch.exp(-2.0 * net["o"][1].abs())
    g = torch.stack([da * 0.95 * s * (1 - s),
                     dk * net["kappa"] * math.log(2.0) * 2.0 * 4.0 * e / (1.0 + e) ** 2])
    gq = _bf(g)
    gh2 = torch.where(net["a2"] > 0, net["w3"].T @ gq, torch.zeros_like(net["a2"]))
    gb = _bf(gh2)
    gh1 = torch.where(net["a1"] > 0, net["w2"].T @ gb, torch.zeros_like(net["a1"]))
    return torch.cat([(_bf(gh1) @ net["x"].T).reshape(-1), gh1.sum(1),
                      (gb @ net["h1"].T).reshape(-1), gh2.sum(1),
                      (gq @ net["h2"].T).reshape(-1), g.sum(1)])


def _xgradient(c, g, alpha):
    """The blend factor raised where the carried samples changed."""
    gr, f32 = c["grad"], torch.float32
    h, w = g.z.shape
    ch, cw = (h + 2) // 3, (w + 2) // 3
    pick = gr["pick"].long()
    qx = 3 * torch.arange(cw, device=DEV)[None, :] + pick % 3
    qy = 3 * torch.arange(ch, device=DEV)[:, None] + pick // 3
    ok = (qx < w) & (qy < h)
    qi = torch.where(ok, qy * w + qx, torch.zeros_like(qx)).reshape(-1)
    ok = ok.reshape(-1)
    at = lambda p: p.reshape(-1)[qi].to(f32)
    px = torch.floor(qx.reshape(-1).to(f32) + at(gr["fmv"][0]) + 0.5)
    py = torch.floor(qy.reshape(-1).to(f32) + at(gr["fmv"][1]) + 0.5)
    ok = ok & (px >= 0) & (px < w) & (py >= 0) & (py < h)
    px, py = px.clamp(0, w - 1).long(), py.clamp(0, h - 1).long()
    zc = g.z.reshape(-1)[py * w + px].to(f32)
    ok = ok & (zc > 0) & torch.isfinite(zc) & ((at(gr["fz"]) - zc).abs() <= 0.1 * zc)
    lum = lambda t: _luma(t.reshape(3, -1)[:, qi].to(D))
    lp, lr = lum(gr["prev"]), lum(gr["reshade"])
    cell = (py // 3) * cw + px // 3
    none = cw * ch
    order = torch.arange(none, device=DEV)
    key = torch.full((none,), none, device=DEV).scatter_reduce(
        0, torch.where(ok, cell, torch.zeros_like(cell)),
        torch.where(ok, order, torch.full_like(order, none)), "amin")
    has = key < none
    key = torch.where(has, key, torch.zeros_like(key))
    p = has.to(D).reshape(ch, cw)
    d = torch.where(has, (lr - lp)[key], 0.0).reshape(ch, cw)
    m = torch.where(has, torch.maximum(lr, lp)[key], 0.0).reshape(ch, cw)
    cy = (3 * torch.arange(ch, device=DEV) + 1).clamp_max(h - 1)
    cx = (3 * torch.arange(cw, device=DEV) + 1).clamp_max(w - 1)
    z, gx, gy = (t[cy][:, cx].to(D) for t in (g.z, g.dzdx, g.dzdy))
    ones = torch.ones_like(z)
    for lvl in range(3):
        s = 1 << lvl
        acc = [torch.zeros_like(z) for _ in range(3)]
        for b in range(-2, 3):
            for a in range(-2, 3):
                dz = (z - _sh(z, a * s, b * s)).abs()
                wt = H5[a + 2] * H5[b + 2] * torch.exp(
                    -dz / ((gx * (3 * a * s) + gy * (3 * b * s)).abs() + 1e-10))
                wt = wt * _sh(ones, a * s, b * s)
                for k, t in enumerate((d, m, p)):
                    acc[k] += wt * _sh(t, a * s, b * s)
        d, m, p = acc
    lam = torch.where((p > 0) & (m > 0), (d.abs() / m.clamp_min(1e-300)).clamp_max(1.0), 0.0)
    lam = lam.repeat_interleave(3, 0).repeat_interleave(3, 1)[:h, :w]
    return alpha + lam * (1.0 - alpha)


def _xcontrol(rough, angle, table):
    one = torch.full(rough.shape if rough is not None else angle.shape, 15, device=DEV)
    if rough is None:
        return torch.where(angle > 6.0, one + 16, one)
    lv = one
    if table:
        lv = torch.where(rough <= 0.0, 0, torch.where(rough <= torch.tensor(0.05), 1, one))
    return torch.where(rough > torch.tensor(0.2), lv + 16, lv)


def exact(case, seed):
    k, half = case["kind"], bool(case.get("half"))
    if k in ("frame", "adaptive", "learned"):
        s, inp, hist, _ = _inputs(case, seed)
        cfg = _config(case)
        net = _network(learn.load_weights()) if k == "learned" else None
        t = _xtemporal(inp, hist, cfg, net=net)
        ctl = None
        if k == "adaptive":
            ctl = _xcontrol(s.rough[s.gbuffer(s.frame)["obj"]], None, True)
        return _xchain(t, inp, cfg, half, kappa=t["kappa"], ctl=ctl)
    if k == "batch":
        outs = []
        for i, c in enumerate(_batch_cases(case)):
            _, inp, hist, _ = _inputs(c, seed + 1000 * i)
            outs.append(_xchain(_xtemporal(inp, hist, MOTION), inp, MOTION, half))
            outs[-1] = {n: v.float() if n in ("out", "rgb") else v for n, v in outs[-1].items()}
        return outs
    if k == "channels":
        c = _channels(case, seed)
        g = c["inp"].g
        alpha = _xgradient(c, g, 0.2)
        shadow = FilterConfig(clamp=True, use_id=True, levels=4)
        spec = FilterConfig(clamp=True, tonemap=True, use_id=True, levels=4)
        streams = []
        for rgb, hist, cfg, am, ctl in (
                (c["shadow"], c["hist"][0], shadow, alpha, _xcontrol(None, c["angle"], False)),
                (c["spec"], c["hist"][1], spec, None, _xcontrol(c["rough"], None, True))):
            inp = FrameInputs(rgb, g, c["inp"].mv, c["inp"].prev)
            streams.append(_xchain(_xtemporal(inp, hist, cfg, alpha=am), inp, cfg, half,
                                   ctl=ctl))
        out = _rounder(half)(c["direct"].to(D) * streams[0]["out"] + streams[1]["out"])
        return dict(out=out, alpha=alpha, streams=streams)
    if k == "train":
        return _xtrain(case, seed)
    if k == "network":
        inp, hist, da, dk = _network_inputs(case, seed)
        t = _xtemporal(inp, hist, MOTION, net=_network(learn.load_weights()))
        grad = _xbackward(t["net"], da.to(D).reshape(-1), dk.to(D).reshape(-1))
        return dict(alpha=t["alpha"], kappa=t["kappa"], grad=grad / da.numel())
    if k == "variance":
        g, m1, m2c, n = _variance_inputs(case, seed)
        return _xvariance(m1.to(D), m2c.to(D), n, _gb(g))
    li = _level_inputs(case, seed)
    out, var = _xlevel(li["c"].to(D), li["v"].to(D), _gb(li["g"]), li["kappa"].to(D),
                       case["step"], case["separable"], _rounder(half))
    return dict(out=_rounder(half)(out), var=var)


def _xtrain(case, seed):
    _, inp, hist, ex = _inputs(case, seed)
    mlp, cfg = learn.load_weights(), MOTION
    t = _xtemporal(inp, hist, cfg, net=_network(mlp))
    g = _gb(inp.g)
    y = ex["clean"].to(D)
    y = y / (1.0 + _luma(y))
    c, v = t["rgb"], _xvariance(t["m1"], t["m2c"], t["n"], g)
    ders = []
    for i in range(cfg.levels):
        c, v = _xlevel(c, v, g, t["kappa"], 1 << i, False, lambda x: x, terms=ders)
    res = (c - y) / (y * y + 0.01)
    on = g["live"] & (t["alpha"] >= 1.0 / t["n"].clamp_min(1).to(D))
    d_alpha = torch.where(on, (2 / 3) * (res * (t["cur"] - t["hist"])).sum(0), 0.0)
    d_kappa = torch.where(g["live"], (2 / 3) * (res * sum(ders)).sum(0), 0.0)
    grad = _xbackward(t["net"], d_alpha.reshape(-1), d_kappa.reshape(-1)) / d_alpha.numel()
    m, v2 = 0.1 * grad, 0.001 * grad * grad
    params = mlp.params.to(D) - 1e-3 * (m / 0.1) / ((v2 / 0.001).sqrt() + 1e-8)
    out = c / (1.0 - _luma(c)).clamp_min(2.0 ** -20)
    return dict(out=out, d_alpha=d_alpha, d_kappa=d_kappa, grad=grad, params=params, m=m, v=v2)
