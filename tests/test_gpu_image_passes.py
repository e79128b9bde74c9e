"""GPU parity of the whole-image passes of a plan against the FP64 oracle at
the edges of their splits: the resolution model (all axes in one pass by 8 x 8
x 8 or 16 x 16 x 1 tiles up to a radius of 4 voxels, one pass per axis
beyond), carried by data updates per event and by image tile, and the prior
update (runs of 2 planes on small images, of 16 on large ones).  Tolerance
as for every iterate."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import img_err, report, smooth_image

pytestmark = pytest.mark.gpu

ITER_TOL = 1e-4


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


def _epoch(P, n, m, seq, beta, fwhm=None, dtv=False):
    """Both sides after the updates seq of a plan of m events in 2 subsets."""
    half = np.asarray(n, dtype=np.float64)
    n_ring = 1 if n[2] == 1 else 6
    sc = lmsynth.Scanner(64, n_ring, 1.3 * float(np.hypot(half[0], half[1])) + 5.0, 2.0 * n[2] / n_ring)
    args = (lmsynth.det_table(sc), 64, n_ring, n, (2.0, 2.0, 2.0), 9, 12.0, 30.0, 3.0, True)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, (2.0, 2.0, 2.0)), lmsynth.TOF(9, 12.0, 30.0, 3.0, True), 1, 1,
                        0.0)
    Gg, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    ev = lmsynth.random_events(p, m, seed=81, min_sep=4)
    s = np.full(m, 0.7, np.float32)
    x0 = smooth_image(Go.shape, 82, base=0.7).astype(np.float32)
    g = (oracle.back(Go, np.ones(m), ev) * 1.1 + 1.0).astype(np.float32)
    gamma = float(np.float32(3.0 / x0.max()))
    cuda = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")
    plan = P.Plan(Gg, Gg.events(ev), cuda(s), 2, gamma, 0.999, beta, g=cuda(g))
    v = smooth_image(Go.shape, 83, base=2.0)
    xi = oracle.dtv_field(v.astype(np.float64), 0.05) if dtv else None
    if dtv:
        plan.set_prior_image(cuda(v), 0.05)
    if fwhm is not None:
        plan.set_resolution(fwhm)
    x = cuda(x0)
    plan.init(x)
    seq = np.asarray(seq, np.int32)
    plan.epoch(x, seq)
    want, st, _ = oracle.lm_spdhg(Go, ev, s.astype(np.float64), g.astype(np.float64), x0, 2, seq, gamma, 0.999, beta,
                                  xi=xi, fwhm=fwhm)
    return img_err(x.cpu().numpy(), want), img_err(plan.get_state()["z"].cpu().numpy(), st.z)


@pytest.mark.parametrize("m", [300, 6000])
@pytest.mark.parametrize("n,fwhm", [
    ((8, 8, 8), (0.7, 0.7, 0.7)),       # exactly one tile, radius 1
    ((9, 7, 17), (1.5, 1.5, 1.5)),      # radius 2
    ((17, 15, 6), (3.1, 0.7, 0.0)),     # radii 4, 1 and an axis left alone
    ((12, 21, 16), (0.0, 2.2, 1.0)),    # radius 3
    ((16, 16, 1), (3.1, 1.5, 0.0)),     # one slice, one tile
    ((33, 15, 1), (0.0, 1.2, 1.2)),     # one slice blurred along z as well
    ((10, 9, 8), (3.2, 1.0, 1.0)),      # radius 5: per axis
])
def test_resolution_model_at_the_edges_of_its_tiles(P, n, fwhm, m):
    ex, ez = _epoch(P, n, m, [0, 2, 1, 1, 2, 0], 0.02, fwhm=fwhm)
    report(f"blur {n} fwhm={fwhm}", events=m, x_err=ex, z_err=ez)
    assert max(ex, ez) <= ITER_TOL


@pytest.mark.parametrize("dtv", [False, True])
@pytest.mark.parametrize("n", [(16, 16, 2), (17, 15, 5), (31, 33, 3), (250, 260, 33)])
def test_prior_update_at_the_edges_of_its_runs(P, n, dtv):
    ex, ez = _epoch(P, n, 4000, [2, 0, 2, 2, 1], 0.02, dtv=dtv)
    report(f"prior {n} dtv={dtv}", x_err=ex, z_err=ez)
    assert max(ex, ez) <= ITER_TOL
