"""Steps with the marker phases beside the collide against every phase in a
launch of its own, bit for bit, where the launches' shapes differ from those of
small lattices: bulk that takes the LDS reservation, bodies whose active planes
are many for each marker workgroup, marker lists in more than the least number
of workgroups, the full-size fish. Several steps in one call, so that each
step's skinning and binning run beside the step before. And both schedules
captured in a graph and replayed, with eager steps in between."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from paper_2206_01683_amd import lbm
from gpu_helpers import say

pytestmark = pytest.mark.gpu

# lattice, storage, body, markers, length or radius, steps
CASES = {
    "fish-192x96x96": ((192, 96, 96), "f32", "fish", 12000, 60.0, 4),
    "fish-203x88x90-bf16": ((203, 88, 90), "bf16", "fish", 6000, 60.0, 4),
    "sphere-192x128x128-r34": ((192, 128, 128), "f32", "sphere", 18000, 34.0, 3),
    "sphere-192x96x96-200000": ((192, 96, 96), "f32", "sphere", 200000, 30.0, 3),
    "sphere-192x128x128-r34-f16": ((192, 128, 128), "f16", "sphere", 18000, 34.0, 3),
    "fish-384x192x192": ((384, 192, 192), "f32", "fish", 12000, 96.0, 3),
}


def _scene(case):
    dims, storage, body, n, length, steps = CASES[case]
    nx, ny, nz = dims
    if body == "fish":
        ms = I.fish_surface(n, length, (0.29 * nx, ny / 2.0, nz / 2.0))
        poses = I.chain_poses(*I.wave_headings(length, 10, np.arange(steps)), ms.joints_rest)
    else:
        ms = I.fibonacci_sphere(n, length, (0.4 * nx, ny / 2.0, nz / 2.0))
        poses = I.identity_poses(steps)
    u = np.array([0.02, 0.0, 0.0])
    frames = I.make_frames(steps, acc=(1e-5, 0.0, 0.0), origin=ms.xrest.mean(axis=1), u_lo=u, u_hi=u)
    return ms, torch.as_tensor(np.ascontiguousarray(poses, np.float32), device="cuda"), frames


def _sim(case, ms, schedule, stream=None):
    (nx, ny, nz), storage = CASES[case][:2]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    u0 = (torch.rand((3, nz, ny, nx), generator=gen, device="cuda") - 0.5) * 4e-3
    u0[0] += 0.02
    torch.cuda.synchronize()
    return lbm.Simulation(nx, ny, nz, 0.6, lbm.BC_VELOCITY, lbm.BC_OUTFLOW, storage=storage, max_markers=ms.n,
                          max_bones=ms.nbones, u0=u0, ib_workgroups=schedule, stream=stream)


@pytest.mark.parametrize("case", list(CASES))
def test_beside_the_collide_matches_launches_of_their_own(case):
    say(f"schedules: {case}")
    ms, poses, frames = _scene(case)
    steps, outs = CASES[case][5], []
    for schedule in (0, -1):
        sim, dm = _sim(case, ms, schedule), lbm.DeviceMarkers(ms)
        wrench = torch.zeros((steps, 8), device="cuda")
        sim.step(frames, dm, poses, wrench)
        torch.cuda.synchronize()
        assert sim.check() == 0
        # the state as stored: after an odd number of steps in the second buffer
        state = sim.fb if steps & 1 else sim.fa
        outs.append([state, dm.F, dm.X, dm.U, wrench])
        sim.close()
    assert float(outs[0][1].abs().max()) > 0
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("schedule", [0, -1])
def test_captured_steps_replay_as_eager_ones(schedule):
    say(f"schedules: graph, schedule {schedule}")
    case = "fish-192x96x96"
    ms, poses, frames = _scene(case)
    steps = CASES[case][5]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, ref = (_sim(case, ms, schedule, stream) for _ in range(2))
        dm, dr = lbm.DeviceMarkers(ms), lbm.DeviceMarkers(ms)
        wrench, want = torch.zeros((steps, 8), device="cuda"), torch.zeros((steps, 8), device="cuda")
        sim.step(frames, dm, poses, wrench)  # both one call on, before the capture
        ref.step(frames, dr, poses, want)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sim.step(frames, dm, poses, wrench)
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
            ref.step(frames, dr, poses, want)
        stream.synchronize()
        for a, b in ((sim.fa, ref.fa), (dm.F, dr.F), (dm.X, dr.X), (wrench, want)):
            assert torch.equal(a, b), f"replay {replay}"
    assert sim.check() == 0 and ref.check() == 0
