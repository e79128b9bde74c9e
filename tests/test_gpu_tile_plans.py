"""GPU parity of plans whose data updates run by image tile, against the FP64
oracle, at the edges of that path: images beyond the tiles that one binning
workgroup counts, images around the number of tiles from which a workgroup has
256 threads instead of 512, plans without TOF and with erfc TOF weights.  That a plan has tile lists is seen from the device memory it
holds, against the same plan in subsets too small for them.  Tolerance as for
every iterate."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import img_err, report
from tests.test_gpu_plan_memory import _USED, _Pool

pytestmark = pytest.mark.gpu

ITER_TOL = 1e-4


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


def _held(P, *args, **kw):
    """A plan and the bytes it holds after its creation."""
    pool = _Pool()
    torch.cuda.synchronize()
    before = pool.get(_USED)
    plan = P.Plan(*args, **kw)
    torch.cuda.synchronize()
    return plan, pool.get(_USED) - before


def _check(P, n, h, tof, subsets, seq, per_tile=4.05, nsigma=3.0):
    half = 0.5 * np.asarray(n) * np.asarray(h)
    sc = lmsynth.Scanner(192, 24, 1.3 * float(np.hypot(half[0], half[1])), 2.0 * half[2] / 24)
    args = (lmsynth.det_table(sc), 192, 24, n, h, 9, 12.0, 30.0, nsigma, tof)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(9, 12.0, 30.0, nsigma, tof), 1, 1, 0.0)
    Gg, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    tiles = int(np.prod([(k + 7) // 8 for k in n]))
    m = int(per_tile * tiles) * subsets + 1
    ev = lmsynth.random_events(p, m, seed=73, min_sep=1)
    s = np.full(m, 0.7, np.float32)
    x0 = np.random.default_rng(74).uniform(0.5, 1.5, Go.shape).astype(np.float32)
    g = (oracle.back(Go, np.ones(m), ev) * 1.1 + 1.0).astype(np.float32)
    gamma = float(np.float32(3.0 / x0.max()))
    evd, sd, gd = Gg.events(ev), torch.as_tensor(s, device="cuda"), torch.as_tensor(g, device="cuda")
    sparse, small = _held(P, Gg, evd, sd, 2 * subsets, gamma, 0.999, 0.02, g=gd)
    sparse.destroy()
    plan, held = _held(P, Gg, evd, sd, subsets, gamma, 0.999, 0.02, g=gd)
    assert held > small + 4 * m, "no tile lists"
    x = torch.as_tensor(x0, device="cuda").clone()
    plan.init(x)
    plan.epoch(x, seq)
    want, _, _ = oracle.lm_spdhg(Go, ev, s.astype(np.float64), g.astype(np.float64), x0, subsets, seq, gamma, 0.999,
                                 0.02)
    e = img_err(x.cpu().numpy(), want)
    report(f"plan by tile {n} tof={tof}", events=m, tiles=tiles, x_err=e)
    assert e <= ITER_TOL


def test_more_tiles_than_one_workgroup_counts(P):
    """40960 tiles, ragged edges: counted in two ranges of tiles."""
    _check(P, (505, 511, 75), (1.0, 1.0, 2.0), True, 2, [0, 1])


@pytest.mark.parametrize("n,tiles,tof,nsigma", [
    ((121, 127, 125), 4096, True, 3.0),   # 256 threads per tile, ragged
    ((121, 113, 123), 3840, True, 3.0),   # 512
    ((111, 97, 40), 910, False, 3.0),     # without TOF
    ((51, 49, 23), 147, True, 24.0),      # a TOF kernel too wide for the table
])
def test_threads_per_tile_and_weights(P, n, tiles, tof, nsigma):
    assert np.prod([(k + 7) // 8 for k in n]) == tiles
    _check(P, n, (2.0, 2.0, 2.0), tof, 2, [0, 2, 1, 2, 0], nsigma=nsigma)
