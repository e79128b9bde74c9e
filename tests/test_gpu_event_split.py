"""GPU parity of the kernels whose split depends on the length of the list or
on the number of image tiles, at the edges of their ranges, against the FP64
oracle: the forward projection (2, 8, 16 or 64 events per wavefront) and the
data update of a plan (512 or 256 threads per 8x8x8 tile), and the projector
pair of lists short enough to work on the caller's image.  Tolerances as for
every projection (1e-5), back projection and iterate (1e-4)."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import img_err, proj_err, report, smooth_image

pytestmark = pytest.mark.gpu

PROJ_TOL = 1e-5
BACK_TOL = 1e-4
ITER_TOL = 1e-4


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


def _geometry(P, n, h, tof, n_cry=96, n_ring=12):
    half = 0.5 * np.asarray(n) * np.asarray(h)
    radius = 1.3 * float(np.hypot(half[0], half[1]))
    n_ring = 1 if n[2] == 1 else n_ring
    sc = lmsynth.Scanner(n_cry, n_ring, radius, 2.0 * half[2] / n_ring if n_ring > 1 else 0.0)
    args = (lmsynth.det_table(sc), n_cry, n_ring, n, h, 9, 12.0, 30.0, 3.0, tof)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(9, 12.0, 30.0, 3.0, tof), 1, 1, 0.0)
    return p, P.Geometry(*args, device="cuda"), oracle.Geometry(*args)


@pytest.mark.parametrize("n,h,tof", [
    ((17, 15, 5), (2.0, 2.6, 3.1), True),
    ((33, 31, 1), (2.0, 2.0, 2.0), True),    # one slice
    ((15, 18, 7), (2.0, 2.0, 2.0), False),   # no TOF: more planes than lanes of an event
])
def test_forward_at_the_edges_of_its_splits(P, n, h, tof):
    p, Gg, Go = _geometry(P, n, h, tof)
    ev = lmsynth.random_events(p, (1 << 19) + 37, seed=61, min_sep=1)
    ev[3], ev[4] = [3, 12, 7, 0, 0], [5, 0, 5, 0, 0]  # no detector, no line: 0
    x = smooth_image(Go.shape, 62)
    xd, evd = torch.as_tensor(x, dtype=torch.float32, device="cuda"), Gg.events(ev)
    first = np.setdiff1d(np.arange(4096), [3, 4])
    for m in (1, 3, (1 << 14) - 1, (1 << 14) + 5, (1 << 16) - 3, (1 << 16) + 17, (1 << 19) - 1, (1 << 19) + 37):
        got = P.lm_fwd(Gg, xd, evd[:m].contiguous()).cpu().numpy()
        assert got.shape == (m,) and np.all(got[3:5] == 0)
        # every length holds the first events; the last ones are its own
        idx = np.concatenate([first, np.arange(m - 4096, m)]) if m >= 8192 else np.arange(m)
        emax, _ = proj_err(got[idx], oracle.fwd(Go, x, ev[idx]))
        report(f"forward split {n} tof={tof}", events=m, err=emax)
        assert emax <= PROJ_TOL


@pytest.mark.parametrize("n,h,tof", [
    ((101, 97, 3), (1.0, 1.3, 1.7), True),
    ((300, 299, 1), (1.0, 1.0, 1.0), False),
])
def test_projector_pair_of_short_lists(P, n, h, tof):
    """Lists short enough to work on the caller's image (by events x planes)
    and lists just beyond, into an image that holds values."""
    p, Gg, Go = _geometry(P, n, h, tof)
    ev = lmsynth.random_events(p, 32767, seed=67, min_sep=1)
    x = smooth_image(Go.shape, 68)
    xd, evd = torch.as_tensor(x, dtype=torch.float32, device="cuda"), Gg.events(ev)
    v = np.random.default_rng(69).uniform(-1, 1, len(ev)).astype(np.float32)
    vd = torch.as_tensor(v, device="cuda")
    for m in (1, 65, 3000, 6000, 9000, 32767):
        got = P.lm_fwd(Gg, xd, evd[:m].contiguous()).cpu().numpy()
        emax, _ = proj_err(got, oracle.fwd(Go, x, ev[:m]))
        img = torch.full(Gg.shape, 0.5, device="cuda")
        P.lm_back(Gg, vd[:m].contiguous(), evd[:m].contiguous(), img)
        want = oracle.back(Go, v[:m].astype(np.float64), ev[:m]) + 0.5
        e = img_err(img.cpu().numpy(), want)
        report(f"short lists {n} tof={tof}", events=m, fwd=emax, back=e)
        assert emax <= PROJ_TOL and e <= BACK_TOL


@pytest.mark.parametrize("n,h,tof", [
    ((25, 23, 17), (2.0, 2.0, 2.0), True),      # 512 threads per tile, ragged
    ((41, 40, 1), (2.0, 2.0, 2.0), False),      # one slice, no TOF
    ((511, 505, 1), (1.0, 1.0, 1.0), True),     # 64 x 64 tiles: 256 threads
    ((503, 512, 1), (1.0, 1.0, 1.0), True),     # 63 x 64 tiles: 512 threads
])
def test_data_update_by_tile(P, n, h, tof):
    """One epoch (two subsets, without and with TV) of a plan with enough
    events per tile for the data update by tile."""
    p, Gg, Go = _geometry(P, n, h, tof, n_cry=128)
    tiles = np.prod([(k + 7) // 8 for k in n])
    m = int(max(4001, 2 * 4 * tiles + 77))
    ev = lmsynth.random_events(p, m, seed=63, min_sep=1)
    s = np.full(m, 0.7, np.float32)
    x0 = np.random.default_rng(64).uniform(0.5, 1.5, Go.shape).astype(np.float32)
    g = oracle.back(Go, np.ones(m), ev) * 1.1 + 1.0
    gamma = float(np.float32(3.0 / x0.max()))
    plan = P.Plan(Gg, Gg.events(ev), torch.as_tensor(s, device="cuda"), 2, gamma, 0.999, 0.02,
                  g=torch.as_tensor(g.astype(np.float32), device="cuda"))
    x = torch.as_tensor(x0, device="cuda").clone()
    plan.init(x)
    seq = lmsynth.subset_sequence(65, 0, 4, 2)
    plan.epoch(x, seq)
    want, _, _ = oracle.lm_spdhg(Go, ev, s.astype(np.float64), g, x0, 2, seq, gamma, 0.999, 0.02)
    e = img_err(x.cpu().numpy(), want)
    report(f"data update by tile {n} tof={tof}", events=m, tiles=int(tiles), x_err=e)
    assert e <= ITER_TOL
