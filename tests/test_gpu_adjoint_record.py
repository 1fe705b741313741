"""A recorded segment whose marker phases run beside the collide against one with
every phase in a launch of its own: states, wrench rows and, through the reverse
sweep (which reads each step's force, macros, lists and records from the ring),
the adjoint state and the pose gradient, bit for bit. Segments of one, two and
five steps, with and without the last state; lattices whose last tiles are one
node wide along an axis, and one periodic along all axes."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from paper_2206_01683_amd import lbm
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nseg,last", [(1, False), (1, True), (2, False), (5, True)])
@pytest.mark.parametrize("dims,open_x", [((33, 24, 25), True), ((24, 17, 20), False)])
def test_record_beside_matches_separate_launches(dims, open_x, nseg, last):
    say(f"record {dims} open={open_x}: {nseg} steps, last state {last}")
    nx, ny, nz = dims
    c, u = (11.0, 8.5, 9.0), np.array([0.02, -0.01, 0.01])
    ms = I.fibonacci_sphere(700, 3.0, c)
    frames = I.make_frames(nseg, acc=(1e-5, 0.0, 0.0), origin=c, u_lo=u, u_hi=u)
    u0 = np.random.default_rng(3).uniform(-0.01, 0.01, (3, nz, ny, nx)).astype(np.float32)
    bc = (I.BC_VELOCITY, I.BC_OUTFLOW) if open_x else (I.BC_PERIODIC, I.BC_PERIODIC)
    poses = torch.as_tensor(I.identity_poses(nseg).astype(np.float32), device="cuda")
    outs = []
    for schedule in (0, -1):
        sim = lbm.Simulation(nx, ny, nz, 0.8, bc[0], bc[1], max_markers=ms.n, max_bones=ms.nbones, u0=u0,
                             with_adjoint=True, ib_workgroups=schedule)
        dm = lbm.DeviceMarkers(ms)
        ckpt = sim.new_state()
        sim.save_state(ckpt)
        states = [torch.zeros_like(ckpt) for _ in range(nseg)]
        ring = states if last else states[:-1] + [None]
        ib_ring, wrench = sim.adjoint_ring(nseg), torch.zeros((nseg, 8), device="cuda")
        sim.adjoint_record(ckpt, ring, dm, poses, frames, ib_ring, wrench)
        rng = np.random.default_rng(5)
        lam = torch.zeros_like(ckpt).view(torch.float32)
        sim.stored_view(lam).copy_(torch.as_tensor(rng.uniform(-1, 1, (27, nz, ny, nx)).astype(np.float32)))
        bar = torch.zeros((nseg, ms.nbones, 24), device="cuda")
        sim.adjoint_segment(ckpt, ring, dm, poses, frames, (1.0, 0.5, -0.3, 0.2), lam, torch.zeros_like(lam), bar,
                            ib_ring, sweep_only=True)
        torch.cuda.synchronize()
        assert sim.check() == 0
        views = [sim.stored_view(s.view(torch.float32)) for s in (states if last else states[:-1])]
        outs.append([t.cpu().numpy().copy() for t in views + [sim.stored_view(lam), bar, wrench]])
        sim.close()
    assert np.abs(outs[0][-2]).max() > 0 and np.abs(outs[0][-1]).max() > 0
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)
