"""Frequency route of periodic cells whose matrices are reduced as Hermitian
ones of order n = 3 N (n <= 192): against the oracle at the edges of the
64-column groups of the reduction (63/66, 126/129, 192) and just past its
range (195: the general reduction of the real embedding), and against the
general reduction itself on a doubled cell, whose eigenvalues at q are those
of the simple cell at the two q points that fold onto it.

Tolerance: the route's 1e-10 Ha per atom.  An eigenvalue carries at most a few
n eps ||K|| = 192 x 2.2e-16 x O(1), a sum over n of them at most n times that
(8e-12 per cell), and the lattice sums are converged to 1e-11 relative."""
import sys

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-10


def _note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


def _run(ctx, c, lattice, qf, coords=None, rep=1, **kw):
    from paper_2308_03140_amd import torch_api as T
    R = c["coords"] if coords is None else coords
    return T.freq_evaluate(ctx, torch.tensor(R, device="cuda"), np.tile(c["alpha0"], rep), np.tile(c["omega"], rep),
                           np.tile(c["rvdw"], rep), beta=c["beta"], a=c["a"], lattice=lattice, q_frac=qf, **kw)


def _compare(N, out, ref, scale=1.0):
    for k in ("energy", "energy_gould"):
        if np.isnan(float(ref[k])):  # a collapsed cell has no logarithm; its other terms still compare
            assert float(ref["min_one_plus_x"]) <= 0.0 and np.isnan(float(out[k]))
            continue
        assert abs(float(out[k]) - scale * float(ref[k])) / N <= TOL, k
    assert abs(float(out["min_one_plus_x"]) - float(ref["min_one_plus_x"])) <= 1e-11
    o, r = (np.asarray(x["orders"].cpu() if hasattr(x["orders"], "cpu") else x["orders"]) for x in (out, ref))
    assert np.abs(o - scale * r[:len(o)]).max() / N <= TOL


@pytest.mark.parametrize("N", [1, 2, 21, 22, 42, 43, 64, 65])
def test_against_oracle(ctx, N):
    _note("freq Hermitian N=%d" % N)
    c = gen.small_crystal(700 + N, N)
    # a generic point and one with a real matrix (no imaginary part in any column)
    qf = np.array([[0.125, -0.375, 0.25], [0.5, 0.0, 0.5]])
    ref = oracle.freq_terms(c["coords"], c["alpha0"], c["omega"], c["rvdw"], c["beta"], c["a"], nfreq=2, norder=4,
                            lattice=c["lattice"], q_frac=qf)
    _compare(N, _run(ctx, c, c["lattice"], qf, n_freq=2, n_order=4), ref)


@pytest.mark.parametrize("N", [33, 40, 64])
def test_folding_against_general_reduction(ctx, N):
    _note("freq Hermitian N=%d against its doubled cell" % N)
    c = gen.small_crystal(800 + N, N)
    lat = np.asarray(c["lattice"], float)
    lat2 = lat.copy()
    lat2[0] *= 2.0
    R2 = np.vstack([c["coords"], c["coords"] + lat[0]])
    a = _run(ctx, c, lat, np.array([[0.125, 0.25, -0.125], [-0.375, 0.25, -0.125]]), n_freq=5, n_order=3)
    b = _run(ctx, c, lat2, np.array([[0.25, 0.25, -0.125]]), coords=R2, rep=2, n_freq=5, n_order=3)
    _compare(2 * N, b, a, 2.0)
