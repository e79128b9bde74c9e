"""How far a voxel that is not finite reaches in a data update by tile: the
events with a sample beside it, and from them the voxels beside their samples
of TOF weight above 0; no other event and no other voxel.  The samples are
those of the projector's definition, with 1e-3 voxels (and mm of the TOF
coordinate) to spare for float32."""
import math

import numpy as np
import pytest
import torch

import lmsynth

pytestmark = pytest.mark.gpu

N, H = (96, 93, 18), (2.0, 2.0, 2.0)
TOF = lmsynth.TOF(9, 12.0, 30.0, 3.0, True)
EPS = 1e-3


def _lines(sc, ev):
    """Per event: dominant axis, the other two, plane range that may be read
    (one plane of margin), and functions of the plane: TOF distance from the
    bin's centre, coordinates along the other axes (voxels)."""
    det = lmsynth.det_table(sc).astype(np.float32)
    p1 = det[ev[:, 0] + sc.n_cry * ev[:, 1].astype(int)]
    p2 = det[ev[:, 2] + sc.n_cry * ev[:, 3].astype(int)]
    d32 = np.abs(p2 - p1)
    a = np.where(d32[:, 1] > d32[:, 0], 1, 0)
    a = np.where(d32[:, 2] > np.maximum(d32[:, 0], d32[:, 1]), 2, a)
    b = np.array([[1, 2], [0, 2], [0, 1]])[a]
    p, d = p1.astype(np.float64), p2.astype(np.float64) - p1
    h, c0 = np.array(H), -0.5 * (np.array(N) - 1) * np.array(H)
    i = np.arange(len(ev))
    lam0, dlam = (c0[a] - p[i, a]) / d[i, a], h[a] / d[i, a]
    dn = np.linalg.norm(d, axis=1)
    half = 3.0 * 30.0 / (2 * math.sqrt(2 * math.log(2))) + 6.0
    tc = 12.0 * ev[:, 4]
    m = (0.5 + (tc[:, None] + np.array([-half, half])) / dn[:, None] - lam0[:, None]) / dlam[:, None]
    lo, hi = np.floor(m.min(1)) - 1, np.ceil(m.max(1)) + 1

    def at(k):
        lam = lam0 + k * dlam
        u = [(p[i, b[:, q]] + lam * d[i, b[:, q]] - c0[b[:, q]]) / h[b[:, q]] for q in range(2)]
        return np.abs((lam - 0.5) * dn - tc), u[0], u[1]
    return a, b, np.maximum(lo, 0), hi, half, at


def test_voxel_that_is_not_finite_reaches_its_samples_only():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    half = 0.5 * np.asarray(N) * np.asarray(H)
    sc = lmsynth.Scanner(192, 12, 1.3 * float(np.hypot(half[0], half[1])), 2.0 * half[2] / 12)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(N, H), TOF, 1, 1, 0.0)
    Gg = P.Geometry(lmsynth.det_table(sc), 192, 12, N, H, 9, 12.0, 30.0, 3.0, True, device="cuda")
    ev = lmsynth.random_events(p, 400_000, seed=71, min_sep=20)
    assert len(ev) // 2 >= 4 * 12 * 12 * 3  # the data update by tile
    plan = P.Plan(Gg, Gg.events(ev), torch.full((len(ev),), 0.7, device="cuda"), 2, 1.0, 0.999, 0.02,
                  g=torch.full(Gg.shape, 50.0, device="cuda"))
    x = torch.full(Gg.shape, 1.0, device="cuda")
    plan.init(x)
    q = np.array([50, 45, 8])
    x[q[2], q[1], q[0]] = math.inf
    plan.epoch(x, [0])
    y = plan.lists()[0].cpu().numpy()
    z = plan.get_state()["z"].cpu().numpy()

    a, b, lo, hi, win, at = _lines(sc, ev)
    k = q[a]
    _, u1, u2 = at(k)
    beside = (np.abs(u1 - q[b[:, 0]]) <= 1 + EPS) & (np.abs(u2 - q[b[:, 1]]) <= 1 + EPS)
    mine = np.arange(len(ev)) % 2 == 0  # subset 0
    may = mine & beside & (k >= lo) & (k <= hi)
    near = mine & beside & (k < lo) & (k >= lo - lo % 4)  # just before the first plane, in its 4-plane group
    assert may.sum() > 20 and near.sum() > 5
    bad = ~np.isfinite(y)
    assert bad.sum() > 10 and not (bad & ~may).any()

    reach = np.zeros(Gg.shape, dtype=bool)
    reach[q[2], q[1], q[0]] = True
    margin = 0  # samples of weight 0 that are on the ray
    for m in range(max(N)):
        t, u1, u2 = at(np.full(len(ev), m))
        inside = bad & (m < np.array(N)[a]) & (m >= lo) & (m <= hi)
        margin += int((inside & (t > win + EPS)).sum())
        for e in np.nonzero(inside & (t <= win + EPS))[0]:
            o = np.zeros(3, dtype=int)
            o[a[e]] = m
            for c1 in range(int(np.floor(u1[e] - EPS)), int(np.floor(u1[e] + EPS)) + 2):
                for c2 in range(int(np.floor(u2[e] - EPS)), int(np.floor(u2[e] + EPS)) + 2):
                    o[b[e, 0]], o[b[e, 1]] = c1, c2
                    if (o >= 0).all() and (o < np.array(N)).all():
                        reach[o[2], o[1], o[0]] = True
    assert margin > 20
    assert np.isfinite(z[~reach]).all()
    assert not np.isfinite(z[reach]).all()
