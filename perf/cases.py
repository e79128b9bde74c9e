"""The work that users of this package have it do, as timed cases.

A case is a dict of plain values.  Every case names a call (`kind`), a
scanner (crystals per ring, rings, radius), an image grid and an event list;
the field of view is fixed per scanner (520 x 520 mm transaxially on the
clinical cylinder, 256 x 256 mm on the single ring), so a grid sets its own
voxel size.  Events are drawn on the GPU from the phantoms of the benchmark
(an ellipsoid with five hot spheres, or a disc with three hot discs) with
smooth contamination, so that lines, tiles and TOF bins carry the uneven
loads of real lists.

`listed` gives the cases, `draw` more of the same ranges, `prepare` what a
user's program holds before the call, `run` one pass through the public
entry points, `work` the bytes and operations a pass cannot do without and
`exact` the same results in 64 bits from plain torch.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2201_05497_amd as P
from paper_2201_05497_amd.autograd import poisson_nll
from paper_2201_05497_amd.serving import Request, solve

DEV = "cuda"
RHO = 0.999
TOF_BIN, TOF_FWHM, TOF_NSIGMA = 24.0, 60.0, 3.0
SIGMA = TOF_FWHM / (2.0 * math.sqrt(2.0 * math.log(2.0)))
SCATTER = 200.0  # mm, width of the contamination's profile

SPHERES = [(80.0 * math.cos(2 * math.pi * j / 5), 80.0 * math.sin(2 * math.pi * j / 5), r)
           for j, r in enumerate((5.0, 7.5, 10.0, 12.5, 15.0))]
DISCS = [(50.0, 0.0, 12.0), (-25.0, 43.3, 16.0), (-25.0, -43.3, 20.0)]


def listed():
    ring = {"n_cry": 360, "n_ring": 1, "nx": 128, "ny": 128, "nz": 1, "tof": True}
    cyl = {"n_cry": 672, "n_ring": 96, "tof": True}
    grid = {"nx": 200, "ny": 200, "nz": 96}        # 2.6 mm voxels
    frame = {"nx": 128, "ny": 128, "nz": 48}       # the dynamic frames' coarser grid
    return [
        # one subset of the single-slice problem: the smallest projection a
        # program asks for, latency and launches
        {"name": "fwd_2d", "kind": "fwd", "events": 3571, **ring},
        # back projection of a short dynamic frame without TOF, an odd grid
        {"name": "back_frame_notof", "kind": "back", "events": 100_003, **cyl, "nx": 121, "ny": 127, "nz": 47,
         "tof": False},
        # one 1e7-event frame, each direction
        {"name": "fwd_3d", "kind": "fwd", "events": 10_000_000, **cyl, **grid},
        {"name": "back_3d", "kind": "back", "events": 10_000_000, **cyl, **grid},
        # a long static scan on the fine grid: forward and back in one pass
        {"name": "pass_long", "kind": "pass", "events": 60_000_000, **cyl, "nx": 300, "ny": 300, "nz": 96},
        # a gradient of the Poisson likelihood over dynamic frames
        {"name": "grad_frames", "kind": "grad", "events": 1_000_000, "frames": 4, **cyl, **frame},
        # LM-SPDHG epochs: the single slice, the 1e7-event reconstruction, and
        # a frame with per-event factors, resolution model and directional TV
        {"name": "epoch_2d", "kind": "epoch", "events": 100_000, "subsets": 28, "prior": "tv", "model": False, **ring},
        {"name": "epoch_3d", "kind": "epoch", "events": 10_000_000, "subsets": 224, "prior": "tv", "model": False,
         **cyl, **grid},
        {"name": "epoch_model", "kind": "epoch", "events": 1_000_000, "subsets": 28, "prior": "dtv", "model": True,
         **cyl, **frame},
        # the warm start of the 1e7-event reconstruction: one EM-TV iteration
        {"name": "emtv_3d", "kind": "emtv", "events": 10_000_000, "subsets": 28, "steps": 20, **cyl, **grid},
        # one request of the reconstruction service, host data in and out
        {"name": "solve_frame", "kind": "solve", "events": 1_000_000, "subsets": 28, "epochs": 3, **cyl, **frame},
        # the sensitivity image of a scanner of 24 rings
        {"name": "sens", "kind": "sens", "n_cry": 384, "n_ring": 24, "nx": 128, "ny": 128, "nz": 24, "tof": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["fwd", "back", "back", "pass", "grad", "epoch", "epoch", "emtv", "solve", "sens"])
    if kind == "sens":
        return {"kind": kind, "n_cry": rng.randint(96, 384), "n_ring": rng.randint(2, 24), "nx": rng.randint(40, 128),
                "ny": rng.randint(40, 128), "nz": rng.randint(5, 24), "tof": rng.random() < 0.8}
    flat = kind in ("fwd", "back", "grad", "epoch") and rng.random() < 0.25
    c = {"kind": kind, "tof": rng.random() < 0.8}
    if flat:
        c.update(n_cry=360, n_ring=1, nx=rng.randint(64, 256), ny=rng.randint(64, 256), nz=1)
    else:
        nx = rng.randint(64, 220)
        c.update(n_cry=672, n_ring=96, nx=nx, ny=max(64, nx + rng.randint(-9, 9)), nz=rng.randint(24, 96))
    if kind in ("fwd", "back"):
        c["events"] = _log(rng, 1_000, 300_000 if flat else 10_000_000 if c["tof"] else 3_000_000)
    elif kind == "pass":
        c["events"] = _log(rng, 1_000_000, 20_000_000)
        c["tof"] = True
    elif kind == "grad":
        c["frames"] = rng.randint(1, 6)
        c["events"] = _log(rng, 2_000, 60_000 if flat else 1_000_000)
    elif kind == "epoch":
        c["events"] = _log(rng, 20_000, 200_000 if flat else 5_000_000)
        c["subsets"] = _log(rng, 4, 56 if flat else 224)
        c["prior"] = rng.choice(["tv", "tv", "dtv"])
        c["model"] = rng.random() < 0.3
    elif kind == "emtv":
        c["events"] = _log(rng, 100_000, 5_000_000)
        c["subsets"] = rng.randint(4, 28)
        c["steps"] = rng.choice([0, 10, 20])
        c["tof"] = True
    else:
        c["events"] = _log(rng, 100_000, 2_000_000)
        c["subsets"] = rng.randint(14, 28)
        c["epochs"] = rng.randint(1, 3)
        c["tof"] = True
    return c


# ---------------------------------------------------------------------------
# scanner, image and event list of a case


class _Setup:
    """Sizes of a case's scanner and grid, and its crystal table."""

    def __init__(self, c):
        self.n_cry, self.n_ring, self.n = c["n_cry"], c["n_ring"], (c["nx"], c["ny"], c["nz"])
        self.flat = self.n_ring == 1
        self.radius, self.pitch = (300.0, 0.0) if self.flat else (380.0, 2.6)
        self.n_tof = 25 if self.flat else 33
        self.kmax = (self.n_tof - 1) // 2
        self.tof = c["tof"]
        fov = 256.0 if self.flat else 520.0
        axial = 2.0 if self.flat else max(1, self.n_ring) * self.pitch
        self.h = (fov / self.n[0], fov / self.n[1], axial / self.n[2])
        self.half_axial = 0.5 * axial
        self.r_img = 0.45 * fov
        phi = 2.0 * np.pi * np.arange(self.n_cry) / self.n_cry
        z = (np.arange(self.n_ring) - (self.n_ring - 1) / 2.0) * self.pitch
        tab = np.empty((self.n_ring, self.n_cry, 3))
        tab[:, :, 0] = self.radius * np.cos(phi)[None]
        tab[:, :, 1] = self.radius * np.sin(phi)[None]
        tab[:, :, 2] = z[:, None]
        self.det = np.ascontiguousarray(tab.reshape(-1, 3).astype(np.float32))

    @property
    def shape(self):
        return (self.n[2], self.n[1], self.n[0])

    @property
    def nvox(self):
        return self.n[0] * self.n[1] * self.n[2]

    def geometry(self):
        return P.Geometry(self.det, self.n_cry, self.n_ring, self.n, self.h, self.n_tof, TOF_BIN, TOF_FWHM,
                          TOF_NSIGMA, self.tof, device=DEV)

    def centres(self, a):
        return (torch.arange(self.n[a], dtype=torch.float64, device=DEV) - (self.n[a] - 1) / 2.0) * self.h[a]

    def n_pairs(self):
        return self.n_cry * (self.n_cry - 1) / 2.0 * self.n_ring ** 2

    def sensitivity(self):
        """A smooth image of the size and level of P^T 1: the chords of all
        pairs of crystals through the field, spread over its voxels, highest
        in the axial centre."""
        th = (np.arange(4000) + 0.5) / 4000 * np.pi
        b = self.radius * np.abs(np.cos(th))
        chord = 2.0 * np.sqrt(np.maximum(self.r_img ** 2 - b * b, 0.0)).mean()
        z = self.centres(2).abs() / self.half_axial
        prof = (1.0 - 0.85 * z) if self.n[2] > 1 else torch.ones_like(z)
        r2 = (self.centres(0)[None, :] ** 2 + self.centres(1)[:, None] ** 2) / (self.r_img ** 2)
        g = prof[:, None, None] * (1.0 + 0.2 * r2)[None]
        inside = (r2 <= 1.0).double()
        scale = self.n_pairs() * chord * (1.0 if self.flat else 0.5) / float((g * inside).sum())
        return (g * scale).to(torch.float32).contiguous()

    def x0(self, trues, g):
        """Uniform activity in a cylinder whose projections add up to the trues."""
        r2 = self.centres(0)[None, :] ** 2 + self.centres(1)[:, None] ** 2
        m = (r2 <= self.r_img ** 2).to(torch.float32).expand(self.shape)
        level = np.float32(trues / float((g.double() * m.double()).sum()))
        return (m * float(level)).contiguous()

    def phantom(self):
        x, y, z = self.centres(0)[None, None, :], self.centres(1)[None, :, None], self.centres(2)[:, None, None]
        if self.flat:
            a = (x ** 2 + y ** 2 + 0 * z <= 100.0 ** 2).double()
            hot = [(x - cx) ** 2 + (y - cy) ** 2 + 0 * z <= r * r for cx, cy, r in DISCS]
        else:
            k = 0.8 * self.half_axial
            a = ((x / 200.0) ** 2 + (y / 150.0) ** 2 + (z / k) ** 2 <= 1.0).double()
            hot = [(x - cx) ** 2 + (y - cy) ** 2 + z ** 2 <= r * r for cx, cy, r in SPHERES]
        for h in hot:
            a = torch.where(h, 4.0, a)
        return a.to(torch.float32).contiguous()


def _points(su: _Setup, m, gen):
    """Emission points of the phantom."""
    u = torch.rand((m, 4), device=DEV, dtype=torch.float32, generator=gen)
    q = 2.0 * u[:, :3] - 1.0
    if su.flat:
        p = torch.stack([100.0 * q[:, 0], 100.0 * q[:, 1], 0 * q[:, 2]], 1)
        act = (p[:, 0] ** 2 + p[:, 1] ** 2 <= 1e4).float()
        for cx, cy, r in DISCS:
            act = torch.where((p[:, 0] - cx) ** 2 + (p[:, 1] - cy) ** 2 <= r * r, 4.0, act)
    else:
        p = q * torch.tensor([200.0, 150.0, 0.8 * su.half_axial], device=DEV)
        act = ((q ** 2).sum(1) <= 1.0).float()
        for cx, cy, r in SPHERES:
            act = torch.where((p[:, 0] - cx) ** 2 + (p[:, 1] - cy) ** 2 + p[:, 2] ** 2 <= r * r, 4.0, act)
    return p, 4.0 * u[:, 3] < act


def _trues(su: _Setup, m, gen):
    """m candidate emissions -> the detected ones as int16 [., 5]."""
    p, keep = _points(su, m, gen)
    d = torch.randn((m, 3), device=DEV, dtype=torch.float32, generator=gen)
    if su.flat:
        d[:, 2] = 0.0
    a = d[:, 0] ** 2 + d[:, 1] ** 2
    b = p[:, 0] * d[:, 0] + p[:, 1] * d[:, 1]
    c = p[:, 0] ** 2 + p[:, 1] ** 2 - su.radius ** 2
    root = torch.sqrt((b * b - a * c).clamp_min(0.0))
    e = [p + ((-b + sgn * root) / a)[:, None] * d for sgn in (1.0, -1.0)]
    lim = su.half_axial if not su.flat else 1e9
    keep &= (e[0][:, 2].abs() <= lim) & (e[1][:, 2].abs() <= lim)
    cry, ring = [], []
    for q in e:
        cry.append(torch.round(torch.atan2(q[:, 1], q[:, 0]) * (su.n_cry / (2 * math.pi))).to(torch.int64) % su.n_cry)
        if su.flat:
            ring.append(torch.zeros_like(cry[-1]))
        else:
            ring.append(torch.round(q[:, 2] / su.pitch + (su.n_ring - 1) / 2.0).clamp(0, su.n_ring - 1).to(torch.int64))
    ln = torch.linalg.vector_norm(e[1] - e[0], dim=1).clamp_min(1.0)
    t = ((p - 0.5 * (e[0] + e[1])) * (e[1] - e[0])).sum(1) / ln
    t = t + SIGMA * torch.randn(m, device=DEV, dtype=torch.float32, generator=gen)
    k = torch.round(t / TOF_BIN).to(torch.int64)
    keep &= (cry[0] != cry[1]) & (k.abs() <= su.kmax)
    return torch.stack([cry[0], ring[0], cry[1], ring[1], k], 1)[keep].to(torch.int16)


def _distance(su: _Setup, ev):
    """Distance of each line of response from the scanner axis."""
    d = math.pi / su.n_cry
    return su.radius * torch.cos((ev[:, 2].float() - ev[:, 0].float()) * d).abs()


def _contam(su: _Setup, m, gen):
    c1 = torch.randint(0, su.n_cry, (m,), device=DEV, generator=gen)
    c2 = (c1 + torch.randint(1, su.n_cry, (m,), device=DEV, generator=gen)) % su.n_cry
    r = torch.randint(0, su.n_ring, (2, m), device=DEV, generator=gen)
    k = torch.randint(-su.kmax, su.kmax + 1, (m,), device=DEV, generator=gen)
    ev = torch.stack([c1, r[0], c2, r[1], k], 1).to(torch.int16)
    keep = torch.rand(m, device=DEV, generator=gen) < torch.exp(-_distance(su, ev) ** 2 / (2 * SCATTER ** 2))
    return ev[keep]


def _events(su: _Setup, n, gen):
    """n prompts in random order, 30 % of them contamination, and its
    expectation per event."""
    n_c = int(round(0.3 * n))
    out = torch.empty((n, 5), dtype=torch.int16, device=DEV)
    at = 0
    for end, make in ((n - n_c, _trues), (n, _contam)):
        while at < end:
            got = make(su, min(8 * (end - at) + 4096, 1 << 23), gen)
            m = min(len(got), end - at)
            out[at:at + m] = got[:m]
            at += m
    step = 1 << 24
    if n <= step:
        out = out[torch.randperm(n, device=DEV, generator=gen)]
    else:  # interleave trues and contamination block by block
        order = torch.argsort(torch.rand(n, device=DEV, generator=gen))
        out = torch.cat([out[order[i:i + step]] for i in range(0, n, step)])
        del order
    th = (np.arange(4000) + 0.5) / 4000 * np.pi
    mean = float(np.exp(-(su.radius * np.cos(th)) ** 2 / (2 * SCATTER ** 2)).mean())
    s0 = n_c / (su.n_pairs() * su.n_tof * mean)
    s = s0 * torch.exp(-_distance(su, out) ** 2 / (2 * SCATTER ** 2))
    return out.contiguous(), s.to(torch.float32).contiguous()


def _inputs(case, seed):
    """The plain inputs of a case, from the seed alone."""
    su = _Setup(case)
    d = {"su": su, "case": case}
    if case["kind"] == "sens":
        # a starting image to add to, as the seed gives it
        gen = torch.Generator(DEV).manual_seed(seed)
        d["g0"] = torch.rand(su.shape, device=DEV, generator=gen)
        return d
    gen = torch.Generator(DEV).manual_seed(seed)
    n, frames = case["events"], case.get("frames", 1)
    evs = [_events(su, n, gen) for _ in range(frames)]
    d["ev"] = torch.cat([e for e, _ in evs]) if frames > 1 else evs[0][0]
    d["s"] = torch.cat([s for _, s in evs]) if frames > 1 else evs[0][1]
    d["g"] = su.sensitivity()
    kind = case["kind"]
    if kind in ("fwd", "back", "pass", "grad"):
        act = su.phantom() * torch.empty((frames,) + su.shape, device=DEV).uniform_(0.5, 1.5, generator=gen)
        d["x"] = (act if frames > 1 else act[0]).contiguous()
        d["v"] = torch.empty(n * frames, device=DEV).uniform_(0.2, 2.0, generator=gen)
    if kind == "grad":
        level = 0.7 * n / float((d["g"].double() * su.phantom().double()).sum())
        d["x"] = (d["x"] * level).contiguous()
    if kind in ("epoch", "emtv", "solve"):
        d["x0"] = su.x0(0.7 * n, d["g"])
        d["gamma"] = float(np.float32(3.0 / float(d["x0"].max())))
        r = random.Random(seed)
        k = case["subsets"]
        d["seq"] = np.array([k if r.random() < 0.5 else r.randrange(k) for _ in range(2 * k * case.get("epochs", 1))],
                            dtype=np.int32)
    if case.get("model"):
        e = d["ev"].float()
        d["m"] = (0.5 + 0.4 * torch.cos(0.23 * (e[:, 0] + e[:, 2])) ** 2).contiguous()
        d["fwhm"] = (4.5 / su.h[0], 4.5 / su.h[1], 4.5 / su.h[2] if su.n[2] > 1 else 0.0)
    if case.get("prior") == "dtv":
        ph = su.phantom()
        d["prior"] = (4.0 - ph).contiguous()
        d["eta"] = 0.03
    return d


BETA = 0.03


def prepare(case, seed):
    d = _inputs(case, seed)
    su, kind = d["su"], case["kind"]
    if kind == "solve":
        d["req"] = Request(geom=su.geometry(), events=d["ev"].cpu().numpy(), s=d["s"].cpu().numpy(),
                           x0=d["x0"].cpu().numpy(), n_subsets=case["subsets"], epochs=case["epochs"], beta=BETA,
                           rho=RHO, gamma=d["gamma"], seq=d["seq"])
        return {"kind": kind, "req": d["req"], "g": d["g"]}
    st = {"kind": kind, "geom": su.geometry(), **{k: d[k] for k in ("ev", "s", "g", "x", "v", "x0", "g0") if k in d}}
    if kind == "grad":
        n = case["events"]
        st["off"] = [n * f for f in range(case["frames"] + 1)]
        st["gf"] = st["g"].expand(st["x"].shape).contiguous()
    if kind == "emtv":
        st.update(subsets=case["subsets"], steps=case["steps"])
    if kind == "epoch":
        plan = P.Plan(st["geom"], st["ev"], st["s"], case["subsets"], d["gamma"], RHO, BETA, g=st["g"])
        if "m" in d:
            plan.set_event_factors(d["m"])
            plan.set_resolution(d["fwhm"])
        if "prior" in d:
            plan.set_prior_image(d["prior"], d["eta"])
        st["x"] = d["x0"].clone()
        plan.init(st["x"])
        st.update(plan=plan, seq=d["seq"])
    return st


def run(st):
    kind = st["kind"]
    if kind == "fwd":
        return P.lm_fwd(st["geom"], st["x"], st["ev"])
    if kind == "back":
        return P.lm_back(st["geom"], st["v"], st["ev"])
    if kind == "pass":
        return P.lm_fwd(st["geom"], st["x"], st["ev"]), P.lm_back(st["geom"], st["v"], st["ev"])
    if kind == "grad":
        x = st["x"].detach().requires_grad_(True)
        loss = poisson_nll(x, st["geom"], st["ev"], st["s"], st["gf"], st["off"])
        loss.backward()
        return {"loss": loss.detach(), "grad": x.grad}
    if kind == "epoch":
        return st["plan"].epoch(st["x"], st["seq"])
    if kind == "emtv":
        return P.lm_emtv(st["geom"], st["ev"], st["s"], st["g"], st["x0"].clone(), st["subsets"], 1, BETA, st["steps"])
    if kind == "solve":
        return solve(st["req"], g=st["g"])
    if kind == "sens":
        return P.lm_sens(st["geom"], st["g0"].clone())
    raise ValueError(kind)


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _samples(su: _Setup):
    """Planes an event visits: its TOF window, or its chord through the field."""
    path = 2 * (TOF_NSIGMA * SIGMA) + TOF_BIN if su.tof else 0.75 * su.n[0] * su.h[0]
    if not su.flat:
        path = min(path, 0.75 * su.n[0] * su.h[0])
    return path / (1.2 * max(su.h[0], su.h[1]))


def work(case):
    su = _Setup(case)
    kind, v = case["kind"], su.nvox
    one = 16.0 * _samples(su)  # operations of one event in one direction: position, weight, four corners
    n = case.get("events", 0) * case.get("frames", 1)
    img = 4 * v * case.get("frames", 1)
    if kind in ("fwd", "back"):
        return {"bytes": 14 * n + img, "flops": one * n}
    if kind == "pass":
        return {"bytes": 28 * n + 2 * img, "flops": 2 * one * n}
    if kind == "grad":
        return {"bytes": 36 * n + 3 * img, "flops": 2 * one * n}
    if kind == "sens":
        chord = 0.6 * su.n[0]
        return {"bytes": 8 * v, "flops": 10.0 * su.n_pairs() * chord}
    k = case["subsets"]
    prior = 44 if case.get("prior", "tv") == "tv" else 56
    # an update reads its events' lists (32 bytes each) and the images it steps
    epoch = {"bytes": 32 * n + k * (28 + prior) * v, "flops": 2 * one * n + 60 * k * v}
    if kind == "epoch":
        if case["model"]:
            epoch = {"bytes": epoch["bytes"] + 32 * k * v, "flops": epoch["flops"] + 60 * k * v}
        return epoch
    if kind == "emtv":
        return {"bytes": 28 * n + k * (16 + 36 * case["steps"]) * v, "flops": 2 * one * n + 40 * k * case["steps"] * v}
    e = case["epochs"]
    return {"bytes": 40 * n + e * epoch["bytes"], "flops": 3 * one * n + e * epoch["flops"]}


# ---------------------------------------------------------------------------
# the same results in 64 bits


class _Projector:
    """The TOF Joseph projector in 64 bits: one sample per image plane across
    a line's dominant axis (the largest difference of its crystals'
    coordinates in float32, the lower axis on ties), bilinear in the plane,
    zero outside the image."""

    def __init__(self, su: _Setup):
        self.su = su
        self.det = torch.as_tensor(su.det, device=DEV)
        dd = dict(dtype=torch.float64, device=DEV)
        self.h = torch.tensor(su.h, **dd)
        self.nn = torch.tensor(su.n, device=DEV)
        self.c0 = torch.tensor([-0.5 * (su.n[a] - 1) * su.h[a] for a in range(3)], **dd)
        self.stride = torch.tensor([1, su.n[0], su.n[0] * su.n[1]], device=DEV)
        self.other = torch.tensor([[1, 2], [0, 2], [0, 1]], device=DEV)

    def chunk(self, total_bins=False):
        planes = max(self.su.n) if (total_bins or not self.su.tof) else 100
        return max(1, (1 << 23) // planes)

    def samples(self, ev, all_bins=False):
        """(first corner's plane index, corners, weights) of a chunk of
        events: index [n, J, 4] (0 where outside), weight [n, J, 4] with the
        line's length factor and TOF weight."""
        su = self.su
        e = ev.to(torch.int64)
        f1, f2 = self.det[e[:, 0] + su.n_cry * e[:, 1]], self.det[e[:, 2] + su.n_cry * e[:, 3]]
        df = (f2 - f1).abs()
        a = torch.zeros(len(e), dtype=torch.int64, device=DEV)
        a = torch.where(df[:, 1] > df[:, 0], 1, a)
        a = torch.where(df[:, 2] > torch.maximum(df[:, 0], df[:, 1]), 2, a)
        p1, d = f1.double(), f2.double() - f1.double()
        pick = lambda t, i: t.gather(1, i[:, None])[:, 0]  # noqa: E731
        da, p1a = pick(d, a), pick(p1, a)
        ok = da != 0
        da = torch.where(ok, da, 1.0)
        b = self.other[a]
        dn = torch.linalg.vector_norm(d, dim=1)
        ha, na = self.h[a], self.nn[a]
        lam0, dlam = (self.c0[a] - p1a) / da, ha / da
        lo, hi = torch.zeros_like(lam0), (na - 1).double()
        la, lb = -lam0 / dlam, (1.0 - lam0) / dlam
        lo, hi = torch.maximum(lo, torch.ceil(torch.minimum(la, lb))), torch.minimum(hi, torch.floor(torch.maximum(la, lb)))
        if su.tof:
            k = 0.0 if all_bins else e[:, 4].double() * TOF_BIN
            half = TOF_NSIGMA * SIGMA + (su.kmax + 0.5 if all_bins else 0.5) * TOF_BIN
            dn1 = dn.clamp_min(1e-9)
            ma, mb = ((0.5 + (k + q * half) / dn1 - lam0) / dlam for q in (-1.0, 1.0))
            lo = torch.maximum(lo, torch.floor(torch.minimum(ma, mb)))
            hi = torch.minimum(hi, torch.ceil(torch.maximum(ma, mb)))
        J = int((hi - lo).max().clamp_min(0).item()) + 1
        m = lo[:, None] + torch.arange(J, device=DEV, dtype=torch.float64)[None]
        live = ok[:, None] & (m <= hi[:, None])
        lam = lam0[:, None] + m * dlam[:, None]
        w = (ha * dn / da.abs())[:, None].expand_as(lam)
        if su.tof:
            t = (lam - 0.5) * dn[:, None]
            half = (su.kmax + 0.5 if all_bins else 0.5) * TOF_BIN
            kc = torch.zeros_like(t) if all_bins else (e[:, 4].double() * TOF_BIN)[:, None]
            vc, sr = TOF_NSIGMA / math.sqrt(2.0), SIGMA * math.sqrt(2.0)
            up = torch.erf(((kc + half - t) / sr).clamp(-vc, vc))
            dn_ = torch.erf(((kc - half - t) / sr).clamp(-vc, vc))
            w = w * (up - dn_) / (2.0 * math.erf(vc))
        w = torch.where(live, w, 0.0)
        base = m.clamp(min=0).to(torch.int64) * self.stride[a][:, None]
        idx, wt = [base], [w]
        for q in range(2):
            ax = b[:, q]
            u = (pick(p1, ax)[:, None] + lam * pick(d, ax)[:, None] - self.c0[ax][:, None]) / self.h[ax][:, None]
            i0 = torch.floor(u)
            f = u - i0
            i0 = i0.clamp(-2, 1 << 20).to(torch.int64)
            n_ax, s_ax = self.nn[ax][:, None], self.stride[ax][:, None]
            ni, nw = [], []
            for c in range(2):
                i = i0 + c
                inside = (i >= 0) & (i < n_ax)
                wc = torch.where(inside, f if c else 1.0 - f, 0.0)
                i = torch.where(inside, i, 0) * s_ax
                for bi, bw in zip(idx, wt):
                    ni.append(bi + i)
                    nw.append(bw * wc)
            idx, wt = ni, nw
        return idx, wt

    def fwd(self, x, ev):
        x = x.double().reshape(-1)
        out = torch.empty(len(ev), dtype=torch.float64, device=DEV)
        for o in range(0, len(ev), self.chunk()):
            idx, wt = self.samples(ev[o:o + self.chunk()])
            acc = sum((x[i.clamp(max=x.numel() - 1)] * w).sum(1) for i, w in zip(idx, wt))
            out[o:o + self.chunk()] = acc
        return out

    def back(self, v, ev, all_bins=False, img=None):
        if img is None:
            img = torch.zeros(self.su.nvox, dtype=torch.float64, device=DEV)
        step = self.chunk(all_bins)
        for o in range(0, len(ev), step):
            idx, wt = self.samples(ev[o:o + step], all_bins)
            for i, w in zip(idx, wt):
                img.index_add_(0, i.clamp(max=img.numel() - 1).reshape(-1), (w * v[o:o + step].double()[:, None]).reshape(-1))
        return img.reshape(self.su.shape)


def _grad(x):
    g = torch.zeros((3,) + x.shape, dtype=x.dtype, device=x.device)
    g[0, :, :, :-1] = x[:, :, 1:] - x[:, :, :-1]
    g[1, :, :-1] = x[:, 1:] - x[:, :-1]
    g[2, :-1] = x[1:] - x[:-1]
    return g


def _adj(w):
    """K^T w."""
    o = torch.zeros(w.shape[1:], dtype=w.dtype, device=w.device)
    o[:, :, :-1] -= w[0, :, :, :-1]
    o[:, :, 1:] += w[0, :, :, :-1]
    o[:, :-1] -= w[1, :, :-1]
    o[:, 1:] += w[1, :, :-1]
    o[:-1] -= w[2, :-1]
    o[1:] += w[2, :-1]
    return o


def _knorm(n):
    return math.sqrt(sum(4.0 * math.sin(math.pi * (k - 1) / (2 * k)) ** 2 for k in n))


def _blur(x, fwhm):
    for ax, f in zip((2, 1, 0), fwhm):
        if f == 0.0:
            continue
        s = f / (2.0 * math.sqrt(2.0 * math.log(2.0)))
        r = math.ceil(3.0 * s)
        w = [math.exp(-t * t / (2.0 * s * s)) for t in range(-r, r + 1)]
        tot, o, n = sum(w), torch.zeros_like(x), x.shape[ax]
        for t, wt in zip(range(-r, r + 1), w):
            a, b = max(0, -t), min(n, n - t)
            if a < b:
                o.narrow(ax, a, b - a).add_(x.narrow(ax, a + t, b - a), alpha=wt / tot)
        x = o
    return x


def _counts(su, ev):
    """Events of each event's sinogram bin (unordered crystals, signed bin)."""
    e = ev.to(torch.int64)
    i, j, k = e[:, 0] + su.n_cry * e[:, 1], e[:, 2] + su.n_cry * e[:, 3], e[:, 4]
    key = (torch.minimum(i, j) * (su.n_cry * su.n_ring) + torch.maximum(i, j)) * su.n_tof + torch.where(i > j, -k, k) + su.kmax
    _, inv, cnt = torch.unique(key, return_inverse=True, return_counts=True)
    return cnt[inv].double()


def _spdhg(d, seq):
    """LM-SPDHG from x0 over the updates of seq."""
    su, case, pr = d["su"], d["case"], _Projector(d["su"])
    ev, s, n = d["ev"], d["s"].double(), case["subsets"]
    g, x, gamma = d["g"].double(), d["x0"].double(), d["gamma"]
    m = d["m"].double() if "m" in d else torch.ones(len(ev), dtype=torch.float64, device=DEV)
    B = (lambda t: _blur(t, d["fwhm"])) if "fwhm" in d else (lambda t: t)
    kn = _knorm(su.n)
    T = RHO / (2.0 * gamma * g.clamp_min(kn))
    Sp = gamma * RHO / kn
    mu = _counts(su, ev)
    # (the floor on P 1 is on the projection without the factors)
    p1 = pr.fwd(B(torch.ones(su.shape, dtype=torch.float64, device=DEV)), ev)
    S = torch.where(p1 > 1e-6 * min(su.h), gamma * RHO / (p1 * m).clamp_min(1e-300), 0.0)
    q = m * pr.fwd(B(x), ev) + s
    y = 1.0 - mu / q
    z = g + B(pr.back(m * (y - 1.0) / mu, ev))
    zbar, w = z.clone(), torch.zeros((3,) + su.shape, dtype=torch.float64, device=DEV)
    xi = None
    if "prior" in d:
        xi = _grad(d["prior"].double())
        xi = xi / torch.sqrt((xi ** 2).sum(0) + d["eta"] ** 2)
    D = (lambda t: t - xi * (xi * t).sum(0)) if xi is not None else (lambda t: t)
    for i in seq:
        x = torch.clamp(x - T * zbar, min=0.0)
        if i < n:
            sl = slice(int(i), None, n)
            e, Se, me, ye, ms = ev[sl], S[sl], mu[sl], y[sl], m[sl]
            v = ye + Se * (ms * pr.fwd(B(x), e) + s[sl])
            yn = 0.5 * (v + 1.0 - torch.sqrt((v - 1.0) ** 2 + 4.0 * Se * me))
            yn = torch.where(Se > 0.0, yn, ye)
            dz = B(pr.back(ms * (yn - ye) / me, e))
            y[sl] = yn
            inv_p = 2.0 * n
        else:
            wn = w + Sp * D(_grad(x))
            wn = wn / (torch.sqrt((wn ** 2).sum(0)) / BETA).clamp_min(1.0)
            dz = _adj(D(wn - w))
            w, inv_p = wn, 2.0
        z = z + dz
        zbar = z + inv_p * dz
    return x


def _emtv(d):
    su, case, pr = d["su"], d["case"], _Projector(d["su"])
    ev, s, g, x, n = d["ev"], d["s"].double(), d["g"].double(), d["x0"].double(), case["subsets"]
    for i in range(n):
        q = pr.fwd(x, ev[i::n]) + s[i::n]
        r = torch.where(q > 0.0, 1.0 / q, 0.0)
        bp = pr.back(r, ev[i::n])
        z = torch.where(g > 0.0, x * n * bp / g, 0.0)
        wt = torch.where(x > 0.0, g / (BETA * x), math.inf)
        u, ub = z.clone(), z.clone()
        p = torch.zeros((3,) + su.shape, dtype=torch.float64, device=DEV)
        gam = float(wt.min())
        gam = gam if math.isfinite(gam) else 0.0
        tau = sig = 1.0 / _knorm(su.n)
        for _ in range(case["steps"]):
            th = 1.0 / math.sqrt(1.0 + 2.0 * gam * tau)
            p = p + sig * _grad(ub)
            p = p / torch.sqrt((p ** 2).sum(0)).clamp_min(1.0)
            un = torch.clamp((u - tau * _adj(p) + tau * torch.where(torch.isinf(wt), 0.0, wt * z)) / (1.0 + tau * wt), min=0.0)
            un = torch.where(torch.isinf(wt), z, un)
            ub, u = un + th * (un - u), un
            tau, sig = tau * th, sig / th
        x = u
    return x


def exact(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    su = d["su"]
    pr = _Projector(su)
    if kind == "fwd":
        return pr.fwd(d["x"], d["ev"])
    if kind == "back":
        return pr.back(d["v"], d["ev"])
    if kind == "pass":
        return pr.fwd(d["x"], d["ev"]), pr.back(d["v"], d["ev"])
    if kind == "grad":
        n, loss, grads = case["events"], 0.0, []
        frames = d["x"].reshape((case["frames"],) + su.shape)
        for f in range(case["frames"]):
            e, x = d["ev"][n * f:n * (f + 1)], frames[f]
            q = pr.fwd(x, e) + d["s"][n * f:n * (f + 1)].double()
            loss = loss + (d["g"].double() * x.double()).sum() - torch.log(q).sum()
            grads.append(d["g"].double() - pr.back(1.0 / q, e))
        return {"loss": loss, "grad": torch.stack(grads) if case["frames"] > 1 else grads[0]}
    if kind == "epoch":
        return _spdhg(d, d["seq"])
    if kind == "solve":
        return _spdhg(d, d["seq"]).cpu().numpy()
    if kind == "emtv":
        return _emtv(d)
    if kind == "sens":
        img = d["g0"].double().reshape(-1)
        c1, c2 = (torch.as_tensor(t, device=DEV) for t in np.triu_indices(su.n_cry))
        r = torch.arange(su.n_ring, device=DEV)
        ra, rb = (t.reshape(-1) for t in torch.meshgrid(r, r, indexing="ij"))
        for o in range(0, len(c1), 128):
            a, b = c1[o:o + 128], c2[o:o + 128]
            e = torch.stack(torch.broadcast_tensors(a[:, None], ra[None], b[:, None], rb[None], torch.zeros_like(ra)[None]), 2).reshape(-1, 5)
            e = e[(e[:, 0] != e[:, 2]) | (e[:, 1] < e[:, 3])]
            pr.back(torch.ones(len(e), device=DEV), e, True, img)
        return img.reshape(su.shape)
    raise ValueError(kind)
