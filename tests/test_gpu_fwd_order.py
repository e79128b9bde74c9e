"""GPU parity of the forward projection from the pair image and in spatial
order against the FP64 oracle: with and without TOF, ragged grids, events that
are out of range or nearly along z, lists just below and above the shortest one
that is ordered.  Tolerance as for every projection; the sums are those of a
list projected in its own order, bit for bit."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import proj_err, report, smooth_image

pytestmark = pytest.mark.gpu

PROJ_TOL = 1e-5
ORDERED = 1 << 19  # events


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


@pytest.mark.parametrize("n,tof", [
    ((181, 179, 65), True),     # in order
    ((101, 97, 55), False),     # in order
    ((65, 63, 30), True),       # pairs in list order
    ((31, 33, 2), True),        # two planes
    ((12, 9, 240), True),       # many rays along z
])
def test_forward_from_pairs_and_in_order(P, n, tof):
    h = (2.0, 2.6, 3.1)
    half = 0.5 * np.asarray(n) * np.asarray(h)
    sc = lmsynth.Scanner(192, 12, 1.3 * float(np.hypot(half[0], half[1])), 2.0 * half[2] / 12)
    args = (lmsynth.det_table(sc), 192, 12, n, h, 9, 12.0, 30.0, 3.0, tof)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(9, 12.0, 30.0, 3.0, tof), 1, 1, 0.0)
    Gg, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    ev = lmsynth.random_events(p, ORDERED + 37, seed=91, min_sep=1)
    bad = np.array([3, 1000, ORDERED + 1])
    ev[bad] = [[192, 0, 3, 0, 0], [3, 12, 7, 0, 0], [-1, 0, 7, 0, 0]]
    ev[5], ev[6] = [5, 0, 5, 3, 0], [5, 0, 5, 0, 0]  # along z; no line
    x = smooth_image(Go.shape, 92)
    xd, evd = torch.as_tensor(x, dtype=torch.float32, device="cuda"), Gg.events(ev)
    for m in (ORDERED - 1, ORDERED + 37):
        got = P.lm_fwd(Gg, xd, evd[:m].contiguous())
        for a in (0, m - 20_000):
            assert torch.equal(P.lm_fwd(Gg, xd, evd[a:a + 20_000].contiguous()), got[a:a + 20_000])
        g = got.cpu().numpy()
        assert np.all(g[bad[bad < m]] == 0) and g[6] == 0
        idx = np.setdiff1d(np.concatenate([np.arange(3000), np.arange(m - 3000, m)]), np.append(bad, 6))
        emax, _ = proj_err(g[idx], oracle.fwd(Go, x, ev[idx]))
        report(f"forward in order {n} tof={tof}", events=m, err=emax)
        assert emax <= PROJ_TOL
