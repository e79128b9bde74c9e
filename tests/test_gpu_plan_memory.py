"""lm_plan_bytes bounds what a plan and its initialisation take from the
device's default memory pool (where the library allocates, and torch does
not): the pool's high-water mark from before lm_plan_create to after
lm_spdhg_init."""
import ctypes

import pytest
import torch

import lmsynth

pytestmark = pytest.mark.gpu

_USED, _USED_HIGH = 7, 8  # hipMemPoolAttrUsedMemCurrent, hipMemPoolAttrUsedMemHigh


class _Pool:
    def __init__(self):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.pool = ctypes.c_void_p()
        assert self.hip.hipDeviceGetDefaultMemPool(ctypes.byref(self.pool), 0) == 0

    def get(self, attr):
        v = ctypes.c_uint64(0)
        assert self.hip.hipMemPoolGetAttribute(self.pool, attr, ctypes.byref(v)) == 0
        return v.value

    def reset_high(self):
        v = ctypes.c_uint64(0)
        assert self.hip.hipMemPoolSetAttribute(self.pool, _USED_HIGH, ctypes.byref(v)) == 0


@pytest.mark.parametrize("n,h,tof,events,subsets,parts,given", [
    ((128, 128, 48), 2.0, False, 1_000_000, 28, 0, True),  # no tile lists: a long list to back project at once
    ((128, 128, 48), 2.0, True, 1_000_000, 224, 4, True),  # small subsets: no tile lists; resolution model
    ((128, 128, 48), 2.0, True, 400_001, 28, 0, True),     # tile lists
    ((64, 63, 1), 2.0, True, 100_003, 4, 0, True),         # one slice
    ((128, 128, 48), 2.0, False, 32_768, 4, 0, True),      # the shortest list that goes by tile
    ((20, 19, 7), 2.0, True, 60_000, 400, 0, False),       # the plan's own sensitivity
    ((20, 19, 7), 2.0, True, 1, 1, 2, True),               # one event; factors
])
def test_plan_and_initialisation_within_plan_bytes(n, h, tof, events, subsets, parts, given):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2201_05497_amd as P
    n_ring = 12 if n[2] > 1 else 1
    sc = lmsynth.Scanner(192, n_ring, 1.1 * h * max(n), h * n[2] / n_ring if n_ring > 1 else 0.0)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, (h,) * 3), lmsynth.TOF(9, 12.0, 30.0, 3.0, tof), 1, 1, 0.0)
    G = P.Geometry(lmsynth.det_table(sc), 192, n_ring, n, (h,) * 3, 9, 12.0, 30.0, 3.0, tof, device="cuda")
    ev = G.events(lmsynth.random_events(p, events, seed=81))
    s, g, x = torch.full((events,), 0.7, device="cuda"), torch.full(G.shape, 50.0, device="cuda"), torch.ones(
        G.shape, device="cuda")
    pool = _Pool()
    torch.cuda.synchronize()
    before = pool.get(_USED)
    pool.reset_high()
    plan = P.Plan(G, ev, s, subsets, 1.0, 0.999, 0.02, g=g if given else None)
    created = pool.get(_USED_HIGH) - before
    if parts & P.PART_FACTORS:
        plan.set_event_factors(torch.ones(events, device="cuda"))
    if parts & P.PART_RESOLUTION:
        plan.set_resolution((2.0, 2.0, 2.0))
    plan.init(x)
    torch.cuda.synchronize()
    high, bound = pool.get(_USED_HIGH) - before, P.lm_plan_bytes(G, events, subsets, parts)
    print(f"[memory] {n} tof={tof} {events}/{subsets}: created {created}, in all {high}, lm_plan_bytes {bound}")
    assert 0 < high <= bound


@pytest.mark.parametrize("n,n_ring,events", [((128, 128, 1), 1, 100_000), ((96, 96, 24), 12, 60_000)])
def test_initialisation_sums_in_double(n, n_ring, events):
    """The batches that fit lm_plan_bytes keep the sums of the back projection
    by tile: z of a new plan against the oracle's, to 1e-6 of its largest value
    (float32 atomics leave 2e-6 and more at these counts)."""
    import numpy as np

    import oracle
    import paper_2201_05497_amd as P
    h = (2.0, 2.0, 2.0)
    sc = lmsynth.Scanner(360, n_ring, 300.0, 2.0 * n[2] / n_ring if n_ring > 1 else 0.0)
    args = (lmsynth.det_table(sc), 360, n_ring, n, h, 25, 24.0, 60.0, 3.0, True)
    p = lmsynth.Problem("t", sc, lmsynth.ImageGeom(n, h), lmsynth.TOF(25, 24.0, 60.0, 3.0, True), 1, 1, 0.0)
    G, Go = P.Geometry(*args, device="cuda"), oracle.Geometry(*args)
    ev = lmsynth.random_events(p, events, seed=83, min_sep=100)
    s = np.full(events, 0.7, np.float32)
    x0 = np.random.default_rng(84).uniform(0.5, 1.5, Go.shape).astype(np.float32)
    g = np.full(Go.shape, 50.0, np.float32)
    plan = P.Plan(G, G.events(ev), torch.as_tensor(s, device="cuda"), 2000, 1.0, 0.999, 0.02,
                  g=torch.as_tensor(g, device="cuda"))
    plan.init(torch.as_tensor(x0, device="cuda"))
    z = plan.get_state()["z"].cpu().numpy().astype(np.float64)
    setup = oracle.lm_setup(Go, ev, 2000, g.astype(np.float64), 1.0, 0.999)
    want = oracle.lm_init(Go, ev, s.astype(np.float64), setup, x0.astype(np.float64)).z
    err = float(np.abs(z - want).max() / np.abs(want).max())
    print(f"[parity] initialisation {n}: z_err={err:.2e}")
    assert err <= 1e-6
