"""The step's marker phases at the sizes where their splits change: the most
markers interpolated straight from the populations and one more (2,000 and
2,001), a marker list longer than the 1,024 entries its workgroup collects in
LDS, markers that fill several stages of 256 records, and periodic axes so short
that a stencil meets a tile from both sides (4 to 18 nodes, last tiles of one and
two nodes). One step from a float32-exact random state against the FP64 oracle:
float32 rounding only, 1e-6 of the population scale; and three steps with the
phases beside the collide against launches of their own, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from gpu_helpers import gpu_run, gpu_sim, interior, oracle_run, random_state, say

pytestmark = pytest.mark.gpu

# nx, ny, nz, markers, radius, centre, open x faces
CASES = {
    "direct-2000": (64, 32, 32, 2000, 6.0, (20.0, 16.0, 16.0), True),
    "macros-2001": (64, 32, 32, 2001, 6.0, (20.0, 16.0, 16.0), True),
    "crowded-1500": (40, 24, 24, 1500, 1.4, (20.5, 12.5, 12.5), True),
    "crowded-3000": (40, 24, 24, 3000, 1.4, (20.5, 12.5, 12.5), True),
    "seams-9x10x17": (9, 10, 17, 60, 1.2, (0.3, 9.8, 16.4), False),
    "seams-4x5x6": (4, 5, 6, 30, 1.0, (3.6, 0.2, 5.5), False),
    "seams-18x8x11": (18, 8, 11, 60, 1.2, (17.7, 7.6, 10.2), False),
    "seams-24x7x33": (24, 7, 33, 60, 1.2, (23.5, 3.0, 32.5), False),
}


def _workload(case):
    nx, ny, nz, n, r, c, open_x = CASES[case]
    ms = I.fibonacci_sphere(n, r, c)
    if not open_x:
        for a, d in enumerate((nx, ny, nz)):
            ms.xrest[a] %= d
    u = np.array([0.02, -0.01, 0.01])
    bc = (I.BC_VELOCITY, I.BC_OUTFLOW) if open_x else (I.BC_PERIODIC, I.BC_PERIODIC)
    return I.Workload(case, nx, ny, nz, 0.8, bc[0], bc[1], 3, np.zeros((3, nz, ny, nx)), ms, I.identity_poses(3),
                      I.make_frames(3, acc=(1e-5, 0.0, 0.0), origin=c, u_lo=u, u_hi=u), np.array([-1.0, 0.0, 0.0]))


@pytest.mark.parametrize("case", list(CASES))
def test_marker_phases_match_oracle_and_separate_launches(case):
    w = _workload(case)
    say(f"step parts: {case}")
    f0 = random_state(w, seed=11)
    ref = oracle_run(w, 1, f0)
    sim, dm, wr = gpu_run(w, 1, f0=f0)
    assert sim.check() == 0
    got = sim.read_populations().cpu().numpy().astype(np.float64)
    err = np.abs(interior(got - ref["f"], w)).max() / np.abs(ref["f"]).max()
    F = dm.F.cpu().numpy()
    ferr = np.abs(F - ref["F"]).max() / np.abs(ref["F"]).max()
    say(f"  populations {err:.2e}, forces {ferr:.2e}, of their largest")
    assert err < 1e-6 and ferr < 1e-5
    outs = []
    for schedule in (0, -1):
        s = gpu_sim(w, f0=f0, ib_workgroups=schedule)
        dev = dm
        poses = torch.as_tensor(w.poses.astype(np.float32), device="cuda")
        wrench = torch.zeros((3, 8), dtype=torch.float32, device="cuda")
        s.step(w.frames, dev, poses, wrench)
        assert s.check() == 0
        outs.append([t.cpu().numpy().copy() for t in (s.read_populations(), dev.F, dev.X, dev.U, wrench)])
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
