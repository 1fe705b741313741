"""Markers that crowd into one tile, at the sizes where the marker lists and the
spreading change: a list that just fills the 4,096 entries that a single lattice
collects in LDS, one more, and several times the 1,024 hits of a plane; in a
batch 1,024 and more. One step from a float32-exact random state against the
FP64 oracle: float32 rounding only, 1e-6 of the population scale and 1e-5 of the
forces'. The spreading adds whole numbers, so that the order of a list, which is
arbitrary, cannot show: the schedules, and the lattices of a batch against lone
runs, agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2206_01683_amd import inputs as I
from paper_2206_01683_amd import lbm
from gpu_helpers import gpu_run, interior, oracle_run, random_state, say

pytestmark = pytest.mark.gpu

DIMS, CENTRE = (40, 24, 24), (20.5, 12.5, 12.5)


def _workload(n, nsteps):
    nx, ny, nz = DIMS
    u = np.array([0.02, -0.01, 0.01])
    return I.Workload(f"crowded-{n}", nx, ny, nz, 0.8, I.BC_VELOCITY, I.BC_OUTFLOW, nsteps, np.zeros((3, nz, ny, nx)),
                      I.fibonacci_sphere(n, 1.4, CENTRE), I.identity_poses(nsteps),
                      I.make_frames(nsteps, acc=(1e-5, 0.0, 0.0), origin=CENTRE, u_lo=u, u_hi=u),
                      np.array([-1.0, 0.0, 0.0]))


@pytest.mark.parametrize("n", [4096, 4097, 9000])
def test_crowded_step_matches_oracle_and_separate_launches(n):
    w = _workload(n, 2)
    say(f"crowded step: {n} markers")
    f0 = random_state(w, seed=11)
    ref = oracle_run(w, 1, f0)
    sim, dm, _ = gpu_run(w, 1, f0=f0)
    assert sim.check() == 0
    got = sim.read_populations().cpu().numpy().astype(np.float64)
    err = np.abs(interior(got - ref["f"], w)).max() / np.abs(ref["f"]).max()
    ferr = np.abs(dm.F.cpu().numpy() - ref["F"]).max() / np.abs(ref["F"]).max()
    say(f"  populations {err:.2e}, forces {ferr:.2e}, of their largest")
    assert err < 1e-6 and ferr < 1e-5
    outs = []
    for schedule in (0, -1):
        s, d, wr = gpu_run(w, 2, f0=f0, ib_workgroups=schedule)
        assert s.check() == 0
        outs.append((s.read_populations().cpu().numpy(), d.F.cpu().numpy(), wr))
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("scheme", [lbm.IB_DIRECT, lbm.IB_IMPLICIT])
def test_crowded_batch_matches_lone_runs(scheme):
    ws = [_workload(n, 3) for n in (1024, 1025, 4500)]
    for w in ws:
        w.ib_scheme, w.mdf_iters = scheme, 2
    want = []
    for w in ws:
        sim, _, wr = gpu_run(w, 3)
        want.append((sim.read_populations().cpu().numpy(), wr))
    for mode in ("phases",) if scheme == lbm.IB_IMPLICIT else ("phases", "persistent"):
        say(f"crowded batch, scheme {scheme}, {mode}")
        b = lbm.Batch(ws, 3)
        b.run(3, mode=mode, graph=False)
        assert b.check() == 0
        with torch.cuda.stream(b.stream):
            got = [s.read_populations() for s in b.sims]
        b.synchronize()
        for j in range(len(ws)):
            np.testing.assert_array_equal(got[j].cpu().numpy(), want[j][0])
            np.testing.assert_array_equal(b.wrench[j].cpu().numpy(), want[j][1])
        b.close()


@pytest.mark.parametrize("n", [1100, 4500])
def test_crowded_record_beside_matches_separate_launches(n):
    say(f"crowded record: {n} markers")
    w = _workload(n, 2)
    f0 = random_state(w, seed=12)
    poses = torch.as_tensor(w.poses.astype(np.float32), device="cuda")
    outs = []
    for schedule in (0, -1):
        sim = lbm.Simulation(*DIMS, 0.8, w.bc_lo, w.bc_hi, max_markers=n, max_bones=1, with_adjoint=True,
                             ib_workgroups=schedule)
        sim.load_populations(f0)
        dm = lbm.DeviceMarkers(w.markers)
        ckpt = sim.new_state()
        sim.save_state(ckpt)
        ring = [torch.zeros_like(ckpt), None]
        ib_ring, wrench = sim.adjoint_ring(2), torch.zeros((2, 8), device="cuda")
        sim.adjoint_record(ckpt, ring, dm, poses, w.frames, ib_ring, wrench)
        lam = torch.zeros_like(ckpt).view(torch.float32)
        seed = np.random.default_rng(5).uniform(-1, 1, (27, DIMS[2], DIMS[1], DIMS[0])).astype(np.float32)
        sim.stored_view(lam).copy_(torch.as_tensor(seed))
        bar = torch.zeros((2, 1, 24), device="cuda")
        sim.adjoint_segment(ckpt, ring, dm, poses, w.frames, (1.0, 0.5, -0.3, 0.2), lam, torch.zeros_like(lam), bar,
                            ib_ring, sweep_only=True)
        torch.cuda.synchronize()
        assert sim.check() == 0
        outs.append([t.cpu().numpy().copy() for t in (sim.stored_view(lam), bar, wrench)])
        sim.close()
    assert np.abs(outs[0][1]).max() > 0
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)
