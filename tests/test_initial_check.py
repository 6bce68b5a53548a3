"""The check of the initial state: the first offending node in order is the one
reported, wherever it lies in the pieces the nodes are scanned in."""
import numpy as np
import pytest

NX, NY = 700, 100   # 70000 nodes: three pieces of 32768, blocks of 512 within


def _check(x0, n):
    from paper_2504_07059_amd import lbm
    diff = [[0.0 if i == j else 0.05 for j in range(n)] for i in range(n)]
    p = lbm.make_params("D2Q9", NX, NY, 1, [1.0, 2.0, 3.0][:n], diff, 1.0,
                        (0.0, 0.0, 0.0), (True, False, False))
    st, _, text = lbm.check_problem(p, x0)
    return text if st else ""


def _x0(n):
    x = np.random.default_rng(n).random((n, NX * NY)) + 0.1
    return x / x.sum(axis=0)


@pytest.mark.parametrize("node", [0, 511, 512, 32767, 32768, 65535, 65536, NX * NY - 1])
@pytest.mark.parametrize("n", [2, 3])
def test_first_offender(node, n):
    good = _x0(n)
    assert _check(good, n) == ""
    for value, text in ((np.nan, "finite"), (-1e-3, "finite"), (np.inf, "finite"),
                        (good[n - 1, node] + 1e-6, "does not sum to 1")):
        x = good.copy()
        x[n - 1, node] = value
        if node + 3 < NX * NY:
            x[0, node + 3] = -1.0      # a later one, not reported
        said = _check(x, n)
        assert text in said
        assert f"node {node} species {n - 1}" in said or said.endswith(f"at node {node}")
    edge = good.copy()
    edge[0, node] += 5e-10             # within the tolerance of the sum
    assert _check(edge, n) == ""
