"""GPU parity of the back projection by image tile (lists of at least 32768
events) against the FP64 oracle:
images around the 16-voxel tile edge, odd and single-slice grids, unequal
voxel sides, with and without TOF, and values that are not finite.
Tolerance as for every back projection: ||gpu - orc||_inf <= 1e-4
||orc||_inf."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import img_err, report

pytestmark = pytest.mark.gpu

BACK_TOL = 1e-4
MIN_LIST = 1 << 15  # lists below this many events go per event


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


def _geometry(P, n, h, tof, n_cry=96, n_ring=12, fwhm=30.0):
    """A cylinder around a box of n voxels of h mm."""
    half = 0.5 * np.asarray(n) * np.asarray(h)
    radius = 1.3 * float(np.hypot(half[0], half[1]))
    n_ring = 1 if n[2] == 1 else n_ring
    pitch = 2.0 * half[2] / n_ring if n_ring > 1 else 0.0
    sc = lmsynth.Scanner(n_cry, n_ring, radius, pitch)
    args = (lmsynth.det_table(sc), n_cry, n_ring, n, h, 9, 12.0, fwhm, 3.0, tof)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(9, 12.0, fwhm, 3.0, tof), 1, 1, 0.0)
    return p, P.Geometry(*args, device="cuda"), oracle.Geometry(*args)


@pytest.mark.parametrize("n,h,tof,fwhm", [
    ((16, 16, 16), (2.0, 2.0, 2.0), True, 30.0),    # exactly one tile
    ((17, 15, 33), (2.0, 2.0, 2.0), True, 30.0),    # one voxel over, one under
    ((37, 29, 11), (2.0, 2.6, 3.1), True, 30.0),    # ragged, unequal sides
    ((40, 40, 5), (1.0, 1.0, 8.0), True, 30.0),     # a z plane spans half a tile of x
    ((33, 47, 1), (2.0, 2.0, 2.0), True, 30.0),     # one slice
    ((48, 31, 20), (2.0, 2.0, 2.0), False, 30.0),   # no TOF
    ((24, 24, 8), (2.0, 2.0, 2.0), True, 400.0),    # TOF kernel too wide for the table: erfc weights
    ((24, 24, 8), (2.0, 2.0, 2.0), True, 3.0),      # bins wider than the truncated kernel
])
def test_back_by_tile_matches_oracle(P, n, h, tof, fwhm):
    p, Gg, Go = _geometry(P, n, h, tof, fwhm=fwhm)
    m = MIN_LIST + 37
    ev = lmsynth.random_events(p, m, seed=51, min_sep=1)
    ev[:5] = [[96, 0, 3, 0, 0], [3, 12, 7, 0, 0], [3, 0, 7, 0, 5], [-1, 0, 7, 0, 0], [5, 0, 5, 0, 0]]
    v = np.random.default_rng(52).uniform(-1, 1, m).astype(np.float32)
    v[::97] = 0.0
    got = P.lm_back(Gg, torch.as_tensor(v, device="cuda"), Gg.events(ev)).cpu().numpy()
    want = oracle.back(Go, v[5:].astype(np.float64), ev[5:])  # the first five contribute nothing
    e = img_err(got, want)
    report(f"back by tile {n} tof={tof} fwhm={fwhm}", events=m, err=e)
    assert e <= BACK_TOL


def test_back_by_tile_accumulates_and_matches_pieces(P):
    """A long list adds to the image that is there, and equals the same list
    in pieces that go per event (both within the back projection tolerance
    of the exact sum)."""
    p, Gg, Go = _geometry(P, (64, 60, 24), (2.0, 2.0, 2.0), True, n_cry=192)
    m = 200_003
    ev = Gg.events(lmsynth.random_events(p, m, seed=53, min_sep=1))
    v = torch.as_tensor(np.random.default_rng(54).uniform(0.2, 2, m).astype(np.float32), device="cuda")
    start = torch.full(Gg.shape, 3.0, device="cuda")
    got = P.lm_back(Gg, v, ev, start.clone())
    ref = start.clone()
    for o in range(0, m, MIN_LIST - 1):
        P.lm_back(Gg, v[o:o + MIN_LIST - 1], ev[o:o + MIN_LIST - 1].contiguous(), ref)
    e = img_err(got.cpu().numpy(), ref.cpu().numpy().astype(np.float64))
    report("back by tile against pieces", events=m, err=e)
    assert e <= 2 * BACK_TOL


def test_back_by_tile_values_that_are_not_finite(P):
    """inf and NaN values reach the voxels that the per-event path gives
    them (corners of weight 0 get nothing), and no others."""
    p, Gg, _ = _geometry(P, (32, 32, 8), (2.0, 2.0, 2.0), True)
    m = MIN_LIST + 5
    ev = lmsynth.random_events(p, m, seed=55, min_sep=1)
    ev[7] = [0, 3, 48, 3, 0]  # along a grid plane's direction: corners of weight 0
    v = np.ones(m, dtype=np.float32)
    v[7], v[100], v[200] = np.inf, -np.inf, np.nan
    evt, vt = Gg.events(ev), torch.as_tensor(v, device="cuda")
    got = P.lm_back(Gg, vt, evt).cpu().numpy()
    ref = P.lm_back(Gg, vt[:MIN_LIST - 1], evt[:MIN_LIST - 1].contiguous())
    ref = P.lm_back(Gg, vt[MIN_LIST - 1:], evt[MIN_LIST - 1:].contiguous(), ref).cpu().numpy()
    assert not np.isfinite(ref).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    assert img_err(got[fin], ref[fin].astype(np.float64)) <= 2 * BACK_TOL
