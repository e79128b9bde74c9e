"""GPU parity of the denoising steps of the listmode EM-TV warm start against
the FP64 oracle at the edges of their split: a workgroup's 64 x 4 columns and
its runs of 4 or 16 planes (16 on large images), odd and even numbers of
steps (the dual and the extrapolated image alternate between two sets of
buffers), and voxels that start at 0.  Tolerance as for every warm start."""
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


@pytest.mark.parametrize("n,steps", [
    ((64, 4, 4), 1),       # one column, one run
    ((65, 7, 5), 2),       # columns of one voxel and of three rows, a run of one plane
    ((63, 9, 16), 3),
    ((1, 17, 9), 5),       # one voxel wide
    ((511, 250, 17), 3),   # runs of 16 planes, the last of one plane
    ((505, 256, 32), 2),
])
def test_denoising_at_the_edges_of_its_split(P, n, steps):
    h = (2.0, 2.0, 2.0)
    radius = 1.3 * float(np.hypot(n[0], n[1])) + 10.0
    sc = lmsynth.Scanner(64, 6, radius, 2.0 * n[2] / 6)
    args = (lmsynth.det_table(sc), 64, 6, n, h, 9, 12.0, 30.0, 3.0, True)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(9, 12.0, 30.0, 3.0, True), 1, 1, 0.0)
    Gg, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    ev = lmsynth.random_events(p, 6000, seed=71, min_sep=8)
    s = np.random.default_rng(72).uniform(0.01, 0.05, len(ev)).astype(np.float32)
    g = (oracle.back(Go, np.ones(len(ev)), ev) * 1.5 + 0.1).astype(np.float32)
    x0 = smooth_image(Go.shape, 73, base=0.5)
    x0[:, 1::5] = 0.0
    x = torch.as_tensor(x0, device="cuda").clone()
    P.lm_emtv(Gg, Gg.events(ev), torch.as_tensor(s, device="cuda"), torch.as_tensor(g, device="cuda"), x, 2, 1, 0.3,
              steps)
    want = oracle.emtv(Go, ev, s.astype(np.float64), g.astype(np.float64), x0.astype(np.float64), 2, 1, 0.3, steps)
    e = img_err(x.cpu().numpy(), want)
    report(f"emtv march {n}", steps=steps, err=e, x_max=float(want.max()))
    assert want.max() > 0 and e <= ITER_TOL
