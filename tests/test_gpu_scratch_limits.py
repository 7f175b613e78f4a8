"""Calls under a workspace limit (MBD_WORKSPACE_LIMIT): from the smallest limit
that a call needs through the diagonalisation alone, it is answered, whichever
route fits, and with the results that it has without a limit.

The limits are bytes, the least that each call ran with before evaluations
formed Q^{-1/2} directly."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _cluster(N):
    return gen.finite_cluster(91, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))


def _args(c, scale=1.0):
    return torch.tensor(c["coords"], device="cuda"), c["alpha0"] * scale, c["omega"], c["rvdw"]


def _answered(monkeypatch, tag, precision, call, least, tol, factors):
    """call(context) -> tensors, under each of the limits and without."""
    from paper_2308_03140_amd import torch_api as T

    def run(limit):
        if limit:
            monkeypatch.setenv("MBD_WORKSPACE_LIMIT", str(int(limit)))
        else:
            monkeypatch.delenv("MBD_WORKSPACE_LIMIT", raising=False)
        ctx = T.Context(0, precision)
        try:
            return [call(ctx) for _ in range(2)]
        finally:
            ctx.close()

    ref = run(None)[0]
    for f in factors:
        print("%s, limit %.2f x %d bytes" % (tag, f, least), flush=True)
        for out in run(f * least):
            assert out.keys() == ref.keys()
            for k in ref:
                assert (out[k] - ref[k]).abs().max().item() <= tol * max(1.0, ref[k].abs().max().item()), (tag, f, k)


# both routes and every order of their sums agree to eps max(8, sqrt(n)) kappa, times four (kappa <= 30 here)
TOL = 4 * 2.2e-16 * 35.0 * 30.0
FACTORS = (1.0, 1.1, 1.5, 2.2, 3.5, 8.0)


@pytest.mark.parametrize("N,least", [(30, 187237), (100, 995186), (400, 12501063)])
def test_energies(monkeypatch, N, least):
    from paper_2308_03140_amd import torch_api as T
    c = _cluster(N)
    for eigvals in (False, True):
        _answered(monkeypatch, "energy of %d atoms, eigvals=%s" % (N, eigvals), "fp64",
                  lambda x: T.evaluate(x, *_args(c), beta=c["beta"], a=c["a"], gradients=False, errors=False,
                                       eigvals=eigvals), least, TOL, FACTORS)


@pytest.mark.parametrize("n,count,dtype,least", [(300, 1, "float64", 986956), (300, 1, "float32", 494239),
                                                 (30, 16, "float64", 1041952)])
def test_eigenvalues(monkeypatch, n, count, dtype, least):
    from paper_2308_03140_amd import torch_api as T
    A = torch.tensor(np.random.default_rng(n).standard_normal((count, n, n)), dtype=getattr(torch, dtype), device="cuda")
    A = A + A.transpose(1, 2)
    _answered(monkeypatch, "eigenvalues %d x %d" % (count, n), "fp64",
              lambda x: {"w": T.eigh(x, A, vectors=False)[0]}, least, 1e-13 if dtype == "float64" else 1e-4, (1.0, 2.0))


@pytest.mark.parametrize("N,least", [(30, 2772359), (150, 32800459)])
def test_frequency_route(monkeypatch, N, least):
    from paper_2308_03140_amd import torch_api as T
    c = _cluster(N)
    _answered(monkeypatch, "frequency route, %d atoms" % N, "fp64",
              lambda x: T.freq_evaluate(x, *_args(c), beta=c["beta"], a=c["a"]), least, 1e-11, (1.0, 2.0))


@pytest.mark.parametrize("n,kgrid,energy,grad", [(3, (1, 2, 2), 802888, 2064487), (8, (2, 2, 2), 1770958, 5399303),
                                                 (24, (2, 2, 1), 3110526, 10931149),
                                                 (40, (2, 2, 2), 9800223, 38624649)])
def test_cells(monkeypatch, n, kgrid, energy, grad):
    from paper_2308_03140_amd import torch_api as T
    c = gen.small_crystal(300 + n, n, kgrid=kgrid)
    kw = dict(beta=c["beta"], a=c["a"], lattice=c["lattice"], kgrid=kgrid, errors=False)
    factors = (1.0, 1.03, 1.06, 1.1, 1.2, 1.35, 1.6, 2.0, 2.6, 3.4, 4.5, 8.0)
    _answered(monkeypatch, "energy of a cell of %d" % n, "fp64",
              lambda x: T.evaluate(x, *_args(c, 0.5), gradients=False, **kw), energy, TOL, factors)
    _answered(monkeypatch, "gradients of a cell of %d" % n, "fp64", lambda x: T.evaluate(x, *_args(c, 0.5), **kw),
              grad, TOL, factors)


@pytest.mark.parametrize("N,least", [(8, 7469), (64, 10623), (256, 15119), (301, 19000)])
def test_pairwise_cells(monkeypatch, N, least):
    """Sums over some 10^5 terms of alternating sign on top of their total; 301
    atoms are more than one round of pairs per workgroup (its limit is an estimate
    of the same rule)."""
    from paper_2308_03140_amd import torch_api as T
    c = gen.small_crystal(300 + N, N, kgrid=(1, 1, 1), side_scale=max(1.0, (N / 40) ** (1 / 3)))
    _answered(monkeypatch, "pairwise energy of a cell of %d" % N, "fp64",
              lambda x: T.ts_evaluate(x, *_args(c), 0.94, lattice=c["lattice"]), least, 1e-12, (1.0, 1.6, 4.0, 100.0))


@pytest.mark.parametrize("precision,N,grad,least", [
    ("fp64", 4, True, 866115), ("fp64", 16, True, 1421146), ("fp64", 60, True, 8620340), ("fp64", 90, True, 19041829),
    ("fp64", 200, True, 74776265), ("fp64", 16, False, 1057665), ("fp64", 90, False, 14922843),
    ("fp32_refined", 16, True, 1375298), ("fp32_refined", 90, True, 20265774), ("fp32_refined", 90, False, 19939388)])
def test_screening(monkeypatch, precision, N, grad, least):
    """The screening's solves carry eps sqrt(n) times the condition of A(u), some
    10^3; FP32 eigenvectors with one refinement step leave up to 10^-6."""
    from paper_2308_03140_amd import torch_api as T
    c = _cluster(N)
    _answered(monkeypatch, "screening of %d atoms, gradients=%s" % (N, grad), precision,
              lambda x: T.rsscs_evaluate(x, *_args(c, 0.5), beta=c["beta"], a=c["a"], gradients=grad, errors=False),
              least, 1e-10 if precision == "fp64" else 2e-6, (1.0, 1.15, 1.5, 2.2, 5.0, 12.0))
