"""Batches where the lookup of an item's environment changes: one wave's compare
and scan reach 64 environments (64, 65 and 130 of them), and odd and even runs,
since consecutive steps alternate between two sets of marker arrays. Lattices of
different small sizes and marker counts (one of them more than the 256 records
that a plane of a tile stages at a time). Bit for bit the lattices run alone,
through the launches with every phase of its own."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from paper_2206_01683_amd import lbm
from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _workload(e, nsteps):
    nx, ny, nz = 20 + e % 5, 17 + e % 3, 16 + e % 4
    c, u = (9.0 + 0.3 * (e % 3), 8.5, 8.0), np.array([0.02, -0.01, 0.01])
    ms = I.fibonacci_sphere(1500 if e == 1 else 40 + e, 1.4 if e == 1 else 3.0, c)
    u0 = np.random.default_rng(e).uniform(-0.01, 0.01, (3, nz, ny, nx))
    return I.Workload(f"env{e}", nx, ny, nz, 0.8, I.BC_VELOCITY, I.BC_OUTFLOW, nsteps, u0, ms,
                      I.identity_poses(nsteps), I.make_frames(nsteps, acc=(1e-5 * e, 0.0, 0.0), origin=c, u_lo=u,
                                                              u_hi=u), np.array([-1.0, 0.0, 0.0]))


@pytest.mark.parametrize("count,nsteps,graph", [(64, 1, False), (65, 3, False), (65, 4, True), (130, 3, False)])
def test_many_environments_match_lone_runs(count, nsteps, graph):
    say(f"batch of {count}, {nsteps} steps, graph={graph}")
    ws = [_workload(e, nsteps) for e in range(count)]
    b = lbm.Batch(ws, nsteps)
    b.run(nsteps, mode="phases", graph=graph)
    assert b.check() == 0
    b.synchronize()
    for e, w in enumerate(ws):
        sim = lbm.Simulation(w.nx, w.ny, w.nz, w.tau, w.bc_lo, w.bc_hi, max_markers=w.markers.n,
                             max_bones=w.markers.nbones, u0=w.u0.astype(np.float32), ib_workgroups=-1)
        wr = torch.zeros((nsteps, 8), device="cuda")
        poses = torch.as_tensor(w.poses[:nsteps].astype(np.float32), device="cuda")
        sim.step(w.frames[:nsteps], lbm.DeviceMarkers(w.markers), poses, wr)
        torch.cuda.synchronize()
        with torch.cuda.stream(b.stream):
            got = b.sims[e].read_populations()
        b.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), sim.read_populations().cpu().numpy())
        np.testing.assert_array_equal(b.wrench[e].cpu().numpy(), wr.cpu().numpy())
