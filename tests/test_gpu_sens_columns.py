"""GPU parity of the sensitivity by transaxial line against the FP64 oracle
at the edges of its split: image planes around the 32 of a wavefront's part,
lines longer than the 64 planes of a chunk, more than 64 and 256 rings, and
TOF bins that cover the field of view wholly, in part or hardly.  Tolerance
as for every back projection."""
import numpy as np
import pytest
import torch

import lmsynth
import oracle
from tests.helpers import img_err, report

pytestmark = pytest.mark.gpu

BACK_TOL = 1e-4


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    return P


@pytest.mark.parametrize("n,n_cry,n_ring,tof,n_tof,tof_bin", [
    ((20, 19, 31), 24, 7, True, 9, 12.0),     # one plane short of a part
    ((20, 19, 32), 24, 7, True, 1, 10.0),     # exactly a part; bins cover little
    ((19, 20, 33), 24, 7, True, 3, 12.0),     # one plane over; bins cover a part
    ((12, 12, 65), 16, 65, False, 1, 12.0),   # 65 rings, three parts
    ((70, 66, 1), 40, 1, True, 9, 12.0),      # two chunks, one slice
    ((9, 10, 8), 10, 258, True, 5, 12.0),     # 258 rings
])
def test_sens_by_line_at_the_edges_of_its_split(P, n, n_cry, n_ring, tof, n_tof, tof_bin):
    h = (2.0, 2.0, 2.0)
    radius = 1.3 * float(np.hypot(n[0], n[1]))
    pitch = 2.0 * n[2] / n_ring if n_ring > 1 else 0.0
    sc = lmsynth.Scanner(n_cry, n_ring, radius, pitch)
    args = (lmsynth.det_table(sc), n_cry, n_ring, n, h, n_tof, tof_bin, 30.0, 3.0, tof)
    Gg, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    want = oracle.sens(Go)
    assert want.max() > 0
    e = img_err(P.lm_sens(Gg).cpu().numpy(), want)
    report(f"sens columns {n} {n_cry}x{n_ring} tof={tof}", err=e)
    assert e <= BACK_TOL
