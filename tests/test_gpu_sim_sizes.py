"""Simulation kernels by matrix size: two-site steps take the smallest kernel
(Jacobi matrices up to 16, 32, 64 or 128) that holds theirs, in a launch
compiled for the largest that the circuit's bonds allow.  Bond caps on both
sides of each line, with truncation, both routings and chain lengths down to
two sites, against the oracle: equal bond dimensions and discarded weights,
fidelity 1 - 1e-10 for circuits without a near-degenerate cut (the bound of
the other simulation tests), and the kernel matrix of the states to 1e-9
(states with a fidelity of 1 - 1e-10 in the worst case differ by ~1e-5 in
amplitude, but measured and expected agreement is at rounding, ~1e-13).
"""
import numpy as np
import pytest

import synthdata as sd
from oracle import gram as ogram
from oracle import mps as omps
from tests.gpu_util import fidelity, require_gpu

pytestmark = pytest.mark.gpu


def _compare(X, d, reps, chi, cutoff, routing, coef=(2.0, 2.0), graph=None):
    import paper_2411_09336_amd as q
    torch = require_gpu()
    spec = q.CircuitSpec(X.shape[1], d, reps, coef[0], coef[1], routing)
    b = q.simulate(torch.tensor(X, device="cuda"), spec, chi, cutoff, graph_circuits=graph)
    assert b.info()["unconverged_svds"] == 0
    dims = b.bond_dims()
    disc, deg = b.trunc_stats()
    ref = [omps.simulate(x, d, reps, chi, cutoff, coef[0], coef[1], routing=routing) for x in X]
    compared = 0
    for i, r in enumerate(ref):
        if r.degenerate_cuts or deg[i]:
            continue
        compared += 1
        assert list(dims[i]) == r.bond_dims
        assert fidelity(b.export(i), r.tensors) > 1 - 1e-10
        assert abs(disc[i] - r.discarded) <= 1e-9 * max(1.0, r.discarded)
    assert compared >= len(X) // 2
    if compared == len(X):
        K = q.gram(b).cpu().numpy()
        assert np.abs(K - ogram.gram([r.tensors for r in ref])).max() < 1e-9
    return dims


@pytest.mark.parametrize("chi", [1, 2, 4, 7, 8, 9, 16, 17, 31, 32, 33, 48])
@pytest.mark.parametrize("routing", [0, 1])
def test_bond_caps(chi, routing):
    X = sd.make_uniform(3, 13, seed=chi)
    dims = _compare(X, 4, 2, chi, 1e-10, routing)
    assert dims.max() <= chi


@pytest.mark.parametrize("m,d", [(2, 1), (3, 2), (4, 3), (5, 1), (70, 1), (70, 2)])
def test_chain_lengths(m, d):
    """Two sites, more sites than waves in a workgroup, and more than the
    lanes of a wave; eager and as graph replays of three circuits."""
    X = sd.make_uniform(5, m, seed=m)
    for graph in (None, 3):
        _compare(X, d, 2, 64, 1e-10, 0, (0.9, 1.3), graph)


def test_bonds_fall_between_gates():
    """Zero angles (features 0 and 1) leave bonds that shrink again, so that
    later steps meet a middle bond above twice its neighbours and clear what
    the larger tensors held."""
    X = sd.make_uniform(4, 12, seed=3)
    X[:, ::3] = 1.0
    X[1, :6] = 1.0
    X[2, 6:] = 1.0
    X[3] = 1.0
    for routing in (0, 1):
        dims = _compare(X, 3, 2, 16, 1e-10, routing)
        assert dims[3].max() == 1
