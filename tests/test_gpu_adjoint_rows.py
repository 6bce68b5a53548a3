"""The reverse step on 3-D lattices wide enough for its 64-column rows: three and
four species take those from 33 columns up (to 64, and from 97 to 128), two species
always, and from 64 columns on a row's last lane reads beyond its wave.  Single
reverse steps against the FP64 oracle and sequences against single steps, to the
bars of the narrower lattices (FP32 arithmetic of the same expressions)."""
import pytest
import torch

from tests import test_gpu_adjoint as A

pytestmark = pytest.mark.gpu

X, Y, Z, NONE = ((True, False, False), (False, True, False), (False, False, True),
                 (False, False, False))


def _case(n, shape, walls, g):
    masses = [1.0, 2.0, 3.0, 5.0][:n]
    return A._wk("d3q19_n%d_%dx%dx%d" % (n, *shape), "D3Q19", shape, masses, walls, g,
                 tuning=dict(block_x=64, rows=2))


CASES = [
    _case(2, (64, 3, 4), X, (2e-5, 0, 0)),
    _case(2, (65, 4, 3), NONE, (1e-5, 2e-6, 0)),
    _case(2, (130, 3, 5), Z, (0, 0, -1e-5)),
    _case(3, (33, 5, 4), Y, (0, 1e-5, 0)),
    _case(3, (64, 4, 5), NONE, (3e-6, 1e-6, 0)),
    _case(3, (100, 3, 4), X, (2e-5, 0, 0)),
    _case(3, (128, 4, 3), Z, (0, 0, 1e-5)),
    _case(4, (40, 3, 4), X, (1e-5, 0, 0)),
    _case(4, (64, 3, 3), Z, (0, 2e-6, -1e-5)),
    _case(4, (127, 4, 3), NONE, (1e-5, 0, 0)),
]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_step_matches_oracle(w):
    A.test_adjoint_step_matches_oracle(w)


# the last three: four population-sized buffers beyond the 256 MB last-level cache,
# whose stores are non-temporal
LARGE = [_case(2, (130, 64, 56), X, (1e-5, 0, 0)), _case(3, (128, 52, 48), Z, (0, 0, 1e-5)),
         _case(4, (64, 80, 52), Y, (0, 1e-5, 0))]
RUNS = [CASES[k] for k in (1, 2, 5, 6, 7, 9)] + LARGE


@pytest.mark.parametrize("w", RUNS, ids=[w.name for w in RUNS])
def test_sequence_equals_single_steps(w):
    A._announce(f"adjoint_run {w.name}")
    sim = A._sim(w)
    n = 4
    s0 = sim.buffers()[0].clone()
    assert (16 * sim.total > 256 << 20) == (w in LARGE)
    seq = torch.zeros((n + 1, (sim.total + 63) // 64 * 64), dtype=torch.float32, device=s0.device)
    seq[0, : sim.total].copy_(s0)
    sim.replay(seq[0], n, seq[1:])
    gen = torch.Generator().manual_seed(9)
    lam = torch.zeros_like(s0)
    sim.view(lam).copy_(torch.randn(tuple(sim.view(s0).shape), generator=gen))
    g_ref = torch.zeros(w.n_species * (w.n_species - 1) // 2 + 3, dtype=torch.float64,
                        device=s0.device)
    a, b = lam.clone(), torch.zeros_like(s0)
    for k in range(n, 0, -1):
        sim.adjoint_step(seq[k - 1, : sim.total], a, b, g_ref)
        a, b = b, a
    got, g = torch.zeros_like(s0), torch.zeros_like(g_ref)
    sim.adjoint_run(seq, n, lam, got, g)
    sim.sync()
    got, ref = sim.view(got), sim.view(a)
    assert (got - ref).abs().max().item() <= 1e-5 * ref.abs().max().item()
    assert (g - g_ref).abs().max().item() <= 1e-5 * g_ref.abs().max().item()
    sim.close()
