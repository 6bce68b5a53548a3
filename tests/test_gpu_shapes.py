"""Execution shapes at the edges of their tiles: every form of the step with one
wave per species (rows, blocks, a persistent grid, and forcing 2 in strips)
against a form that takes every shape: one thread per column in 2-D, the blocks
narrower than a wave in 3-D.  The forms evaluate the same expressions in the same
order, so states and fields agree to the bit (in 3-D the compiler fuses
multiplications and additions of the one-thread form differently, so forms of one
variant are compared there); the sums of the observables, FP64 over at most 2^16
terms in another order, to 2^16 * 2^-53 < 1e-11 relative to the sum of magnitudes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MASSES = [1.0, 2.0, 3.0, 4.0]
PAIRS = {(0, 1): 0.0335, (0, 2): 0.0369, (0, 3): 0.0833, (1, 2): 0.0183, (1, 3): 0.0640,
         (2, 3): 0.0756}


def _sim(dims, n, walls, forcing, field, tuning):
    from paper_2504_07059_amd import lbm
    nx, ny, nz = dims
    diff = [[PAIRS.get((min(i, j), max(i, j)), 0.0) for j in range(n)] for i in range(n)]
    g = (0.0, 0.0, 0.0) if field else (1e-5, -2e-5, 1e-5 if nz > 1 else 0.0)
    p = lbm.make_params("D3Q19" if nz > 1 else "D2Q9", nx, ny, nz, MASSES[:n], diff, 1.0, g,
                        walls, forcing=forcing)
    rng = np.random.default_rng(nx + 1000 * ny + n)
    x0 = rng.random((n, nz, ny, nx)) + 0.2
    x0 /= x0.sum(axis=0)
    accel = None
    if field:
        d = 3 if nz > 1 else 2
        accel = torch.as_tensor(1e-5 * rng.standard_normal((d, nz, ny, nx)), dtype=torch.float32,
                                device="cuda")
    sim = lbm.LbmMc(p, x0, accel=accel)
    sim.set_tuning(*tuning)
    return sim


def _run(*args):
    sim = _sim(*args)
    sim.step(3)
    m = sim.moments(velocities=True)
    raw = sim.raw().clone()
    sim.sync()
    return raw, m


X, Y, Z, XY, NONE = ((True, False, False), (False, True, False), (False, False, True),
                     (True, True, False), (False, False, False))

# dims, species, walls, forcing, force field, shapes (bx, by, rows, persistent, split)
ROWS = [(64, 1, 1, 0, 1), (64, 1, 3, 0, 1), (64, 1, 16, 0, 1), (64, 1, 2, 3, 1)]
CASES = [
    # 2-D rows around one and two waves; three layers, the least between walls
    ((3, 3, 1), 2, XY, 0, False, ROWS),
    ((63, 7, 1), 3, X, 1, False, ROWS),
    ((64, 5, 1), 4, Y, 0, True, ROWS),
    ((65, 9, 1), 2, NONE, 1, False, ROWS),
    ((129, 6, 1), 3, XY, 0, False, ROWS),
    # forcing 2 in strips: one strip, lanes beyond it, two and four uneven
    # strips, the narrowest lattices; and widths that keep the pre-pass
    ((3, 3, 1), 2, XY, 2, False, ROWS),
    ((1, 4, 1), 3, NONE, 2, False, ROWS),
    ((2, 5, 1), 2, Y, 2, False, ROWS),
    ((61, 3, 1), 3, Y, 2, False, ROWS),
    ((62, 4, 1), 4, X, 2, False, ROWS),
    ((64, 4, 1), 3, X, 2, False, ROWS),
    ((65, 8, 1), 2, X, 2, True, ROWS),
    ((124, 11, 1), 3, XY, 2, False, ROWS),
    ((125, 11, 1), 3, NONE, 2, False, ROWS),
    ((249, 13, 1), 4, XY, 2, False, ROWS),
    ((250, 2, 1), 2, X, 2, True, ROWS),
    # 3-D: blocks of rows, and blocks narrower than a wave
    ((5, 4, 3), 2, Z, 0, False, ROWS + [(16, 4, 1, 0, 1)]),
    ((66, 3, 4), 3, X, 1, False, ROWS + [(64, 2, 2, 0, 1)]),
    ((40, 5, 6), 4, Y, 2, False, ROWS),
]


@pytest.mark.parametrize("dims,n,walls,forcing,field,shapes", CASES,
                         ids=["%dx%dx%d-n%d-f%d" % (*c[0], c[1], c[3]) for c in CASES])
def test_shapes_agree(dims, n, walls, forcing, field, shapes):
    print(f"\n[gpu case] shapes {dims} n={n} forcing={forcing}", flush=True)
    form = (64, 1, 2, 0, 0) if dims[2] == 1 else (32, 2, 2, 0, 1)
    ref, mref = _run(dims, n, walls, forcing, field, form)
    assert torch.isfinite(ref).all()
    scale = {"mass": mref["mass"], "momentum": float(mref["rho"].sum())}
    for shape in shapes:
        got, m = _run(dims, n, walls, forcing, field, shape)
        assert torch.equal(got, ref), shape
        for k in ("rho", "x", "u", "ueq", "us"):
            assert torch.equal(m[k], mref[k]), (shape, k)
        for k in ("mass", "momentum"):
            assert np.all(np.abs(m[k] - mref[k]) <= 1e-11 * scale[k]), (shape, k)
