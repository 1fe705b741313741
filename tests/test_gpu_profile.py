"""The measurement hook: every step is counted, and its two parts are what the
header says. In launches of their own the immersed-boundary kernels take time in
every step; beside the collide only a call's first step has anything before it."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from paper_2206_01683_amd import lbm

pytestmark = pytest.mark.gpu


def _parts(schedule, calls, steps):
    w = I.sphere_workload(nsteps=steps)
    sim = lbm.Simulation(w.nx, w.ny, w.nz, w.tau, w.bc_lo, w.bc_hi, max_markers=w.markers.n, u0=w.u0.astype(np.float32),
                         max_bones=w.markers.nbones, ib_workgroups=schedule)
    dm = lbm.DeviceMarkers(w.markers)
    poses = torch.as_tensor(w.poses[:steps].astype(np.float32), device="cuda")
    sim.step(w.frames[:steps], dm, poses)  # not timed: the kernels are loaded on the first call
    sim.profile()
    for _ in range(calls):
        sim.step(w.frames[:steps], dm, poses)
    got, again = sim.profile_collect(), sim.profile_collect()
    sim.close()
    assert again == (0.0, 0.0, 0)
    return got


def test_parts_and_counts():
    own, one, many = _parts(-1, 3, 8), _parts(0, 24, 1), _parts(0, 3, 8)
    for ib, collide, n in (own, one, many):
        assert n == 24 and ib > 0.0 and collide > 0.0
    # 24 steps: skinning and binning before each of 24 calls, or of 3
    assert many[0] < 0.5 * one[0]
    # in launches of their own all the phases count, not those two alone
    assert own[0] > one[0]
