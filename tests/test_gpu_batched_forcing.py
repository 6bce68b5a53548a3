"""The whole corrected forcing on a batch of uneven 2-D tubes, which runs in strips:
every lattice as in its run alone, to the bit (the forms of the step evaluate the
same expressions in the same order), in one launch and in one per lattice."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

X, XY = (True, False, False), (True, True, False)
TUBES = [(61, 7, X), (65, 3, XY), (249, 12, X), (125, 5, XY), (130, 31, X), (300, 4, XY)]
MASSES = [1.0, 2.0, 3.0]
DIFF = [[0.0, 0.0335, 0.0369], [0.0335, 0.0, 0.0183], [0.0369, 0.0183, 0.0]]


@pytest.mark.parametrize("one_launch", [1, 0])
@pytest.mark.parametrize("field", [False, True])
def test_batch_equals_single_runs(one_launch, field):
    from paper_2504_07059_amd import lbm
    print(f"\n[gpu case] forcing 2 batch one_launch={one_launch} field={field}", flush=True)
    strips = sum((nx + 61) // 62 * ny for nx, ny, _ in TUBES)
    tiles = sum((nx + 63) // 64 * ny for nx, ny, _ in TUBES)
    assert 3 * strips < 4 * tiles   # few enough strips for the one-pass form
    params, x0, accel = [], [], []
    for k, (nx, ny, walls) in enumerate(TUBES):
        g = (0.0, 0.0, 0.0) if field else (1e-5, -2e-5 * k, 0.0)
        params.append(lbm.make_params("D2Q9", nx, ny, 1, MASSES, DIFF, 1.0, g, walls,
                                      forcing="full"))
        rng = np.random.default_rng(k)
        x = rng.random((3, nx * ny)) + 0.2
        x0.append((x / x.sum(axis=0)).reshape(-1))
        accel.append(torch.as_tensor(1e-5 * rng.standard_normal(2 * nx * ny),
                                     dtype=torch.float32, device="cuda"))
    sim = lbm.LbmMc(params, np.concatenate(x0), accel=torch.cat(accel) if field else None)
    sim.set_batched_mode(one_launch)
    sim.step(9)
    out = sim.moments(velocities=True)
    sim.sync()
    for l, p in enumerate(params):
        one = lbm.LbmMc(p, x0[l], accel=accel[l] if field else None)
        one.step(9)
        m = one.moments(velocities=True)
        one.sync()
        assert torch.equal(sim.raw("cur", l), one.raw("cur")), TUBES[l]
        for k in ("rho", "x", "u"):
            assert torch.equal(sim.field(out, k, l), one.field(m, k)), (TUBES[l], k)
        one.close()
    sim.close()
