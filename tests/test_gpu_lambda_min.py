"""lambda_min of evaluations without eigenvalues (Lanczos run on powers of
Q^{-1/2}, more squarings the smaller the work) against the diagonalisation:
orders on both sides of each number of squarings, batches and cells, and
spectra whose lowest eigenvalue stands far below the others, where the powers
are close to rank one.

Tolerance: an eigenvalue at the lower end carries eps sqrt(n) kappa relative
of rounding from either route (the bound that the tests of the root use, four
times that), kappa = lambda_max / lambda_min."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("coords", "alpha0", "omega", "rvdw")


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


def _cluster(N, seed=0):
    return gen.finite_cluster(4100 + N + seed, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))


def _eval(ctx, c, **kw):
    from paper_2308_03140_amd import torch_api as T
    a = [torch.tensor(c[k], dtype=torch.float64, device="cuda") for k in KEYS]
    return T.evaluate(ctx, *a, beta=c["beta"], a=c["a"], **kw)


def _check(low, w, tag):
    w = w.flatten().double()
    lo, kappa, n = w.min().item(), (w.max() / w.min()).item(), w.numel()
    tol = 4 * 2.2e-16 * max(8.0, n ** 0.5) * kappa
    assert abs(low - lo) <= tol * lo, (tag, low, lo, tol)


@pytest.mark.parametrize("N", [1, 2, 4, 21, 22, 64, 65, 85, 86, 300, 490, 560, 640, 690, 760, 800])
def test_orders(ctx, N):
    print("lambda_min N=%d" % N, flush=True)
    c = _cluster(N)
    _check(_eval(ctx, c, gradients=False)["errors"][0].item(),
           _eval(ctx, c, gradients=False, eigvals=True)["eigvals"], N)


@pytest.mark.parametrize("N", [12, 50, 64, 100, 320])
def test_isolated(ctx, N):
    """Two atoms close together push one eigenvalue far below the rest."""
    c = _cluster(N)
    X, al = np.array(c["coords"]), np.array(c["alpha0"])
    X[:2] += 400.0
    for ratio in (0.5, 0.9, 0.99, 0.9999):
        print("lambda_min N=%d, pair at %g of the collapse" % (N, ratio), flush=True)
        # along the axis lambda = omega^2 (1 - 2 alpha f / r^3); f is close to 1 at beta = 0.05
        X[1] = X[0] + np.array([0.0, 0.0, 8.0])
        om = np.array(c["omega"])
        om[:2] = 0.5
        al[:2] = ratio * 8.0 ** 3 / 2
        cc = dict(c, coords=X, alpha0=al, omega=om, beta=0.05)
        try:
            w = _eval(ctx, cc, gradients=False, eigvals=True)["eigvals"]
        except Exception as e:  # the damping leaves a collapse: the other route reports it too
            with pytest.raises(type(e)):
                _eval(ctx, cc, gradients=False)
            continue
        _check(_eval(ctx, cc, gradients=False)["errors"][0].item(), w, (N, ratio))


@pytest.mark.parametrize("count,nmin,nmax", [(5, 3, 40), (60, 5, 90), (300, 10, 300)])
def test_batches(ctx, count, nmin, nmax):
    from paper_2308_03140_amd import torch_api as T
    print("lambda_min batch of %d" % count, flush=True)
    mols = [_cluster(int(N), i) for i, N in enumerate(np.random.default_rng(count).integers(nmin, nmax + 1, count))]
    for rep in range(2):
        outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
        for i in range(0, count, max(1, count // 20)):
            assert outs[i]["status"] == 0
            _check(outs[i]["errors"][0].item(), _eval(ctx, mols[i], gradients=False, eigvals=True)["eigvals"], i)


@pytest.mark.parametrize("n,k", [(3, (1, 2, 2)), (8, (2, 2, 2)), (11, (2, 1, 1)), (43, (2, 1, 1)), (64, (2, 2, 2))])
def test_cells(ctx, n, k):
    from paper_2308_03140_amd import torch_api as T
    print("lambda_min cell of %d" % n, flush=True)
    c = gen.small_crystal(300 + n, n, kgrid=k)
    a = [torch.tensor(np.array(c[q]) * (0.5 if q == "alpha0" else 1.0), dtype=torch.float64, device="cuda") for q in KEYS]
    run = lambda **kw: T.evaluate(ctx, *a, lattice=c["lattice"], kgrid=k, beta=c["beta"], a=c["a"], gradients=False, **kw)
    _check(run()["errors"][0].item(), run(eigvals=True)["eigvals"], n)
