"""Q^{-1/2} without eigenvectors (the route of every evaluation that does not
ask for eigenvalues) against the diagonalisation (eigvals=True) on the same
inputs: orders at the edges of the tiles and of the kernels' ranges, spectra
from narrow to beyond the range of the method's table, batches that mix them,
and workspace limits that only one of the two routes fits."""
import sys

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("energy", "grad_coords", "grad_alpha0", "grad_omega", "grad_rvdw")


def _note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


def _cluster(seed, N):
    return gen.finite_cluster(seed, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))


def _run(ctx, c, **kw):
    from paper_2308_03140_amd import torch_api as T
    return T.evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"],
                      beta=c["beta"], a=c["a"], **kw)


def _same(a, b, n, kappa=30.0):
    """Both routes work in FP64: an element of Q^{-1/2} carries about
    eps sqrt(n) of rounding times the conditioning of the root."""
    tol = 2.2e-16 * max(8.0, n ** 0.5) * kappa * 4.0
    # dE/domega is a difference of terms near 3/2
    scale = {k: max(1.0 if k == "grad_omega" else 1e-3, a[k].abs().max().item()) for k in KEYS}
    scale["energy"] = 0.5 * n
    for k in KEYS:
        err = (a[k] - b[k]).abs().max().item()
        assert err <= tol * scale[k], (k, err, tol * scale[k])
    if "errors" in b:
        la, lb = a["errors"][0].item(), b["errors"][0].item()
        assert abs(la - lb) <= 1e-15 * n ** 0.5 * 10 + 1e-12 * abs(la)


@pytest.mark.parametrize("N", [1, 2, 3, 10, 11, 20, 21, 22, 42, 43, 85, 86, 128, 149, 150, 171, 256, 341, 342, 682, 683])
def test_orders(ctx, N):
    _note("direct root N=%d" % N)
    c = _cluster(700 + N, N)
    _same(_run(ctx, c, eigvals=True), _run(ctx, c), 3 * N)
    # without lambda_min, and without gradients
    e = _run(ctx, c, errors=False, gradients=False)["energy"].item()
    assert abs(e - _run(ctx, c)["energy"].item()) <= 1e-14 * 3 * N


def _scaled_to(ctx, c, ratio):
    """alpha0 scaled until lambda_min / lambda_max = ratio (bisection on the
    diagonalisation's eigenvalues)."""
    lo, hi = 0.2, 3.0
    for _ in range(50):
        s = 0.5 * (lo + hi)
        try:
            w = _run(ctx, dict(c, alpha0=c["alpha0"] * s), eigvals=True, gradients=False)["eigvals"][0]
            r = (w[0] / w[-1]).item()
        except Exception:
            r = -1.0
        lo, hi = (s, hi) if r > ratio else (lo, s)
    return dict(c, alpha0=c["alpha0"] * lo)


@pytest.mark.parametrize("N", [12, 40, 160])
def test_spectra(ctx, N):
    """lambda_max/lambda_min through every class of the table and beyond it
    (where the diagonalisation answers)."""
    c = _cluster(40 + N, N)
    for kappa in (20, 40, 90, 180, 400, 900, 3000, 20000):
        cc = _scaled_to(ctx, c, 1.0 / kappa)
        _note("direct root N=%d kappa %g" % (N, kappa))
        _same(_run(ctx, cc, eigvals=True), _run(ctx, cc), 3 * N, kappa=float(kappa))


def test_weakly_coupled_identical_atoms(ctx):
    """Q close to a multiple of the identity: the Lanczos recurrence ends at
    once or runs on couplings near rounding."""
    g = np.array([[i, j, 0] for i in range(6) for j in range(5)], float)
    for spacing in (12.0, 60.0, 3000.0):
        _note("direct root, identical atoms %g bohr apart" % spacing)
        n = len(g)
        c = {"coords": g * spacing, "alpha0": np.full(n, 20.0), "omega": np.full(n, 0.5), "rvdw": np.full(n, 3.5),
             "beta": 0.83, "a": 6.0}
        _same(_run(ctx, c, eigvals=True), _run(ctx, c), 3 * n)


def test_batch_mixed(ctx):
    """One batch of narrow, wide and collapsed spectra and tiny systems: each
    member as on its own, on the eager call and on the replay."""
    from paper_2308_03140_amd import torch_api as T
    _note("direct root, mixed batch")
    base = [_cluster(81, 40), _cluster(82, 7), _cluster(83, 100), _cluster(84, 1), _cluster(85, 23)]
    wide = [_scaled_to(ctx, base[0], 1e-3), _scaled_to(ctx, base[4], 1e-5)]
    bad = dict(base[1], coords=np.array([[0.0, 0, 0], [0, 0, 3.0]]), alpha0=np.array([200.0, 200.0]),
               omega=np.array([0.5, 0.5]), rvdw=np.array([1.0, 1.0]), beta=0.0)
    mols = base + wide + [bad]
    single = [_run(ctx, m, eigvals=True) for m in mols[:-1]]
    for rep in range(3):
        outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
        assert [o["status"] for o in outs] == [0] * (len(mols) - 1) + [2]
        for m, o, s in zip(mols, outs, single):
            n = 3 * len(m["omega"])
            kappa = (s["eigvals"][0][-1] / s["eigvals"][0][0]).item()
            _same(s, dict(o, grad_rvdw=s["grad_rvdw"]), n, kappa=max(30.0, kappa))


def test_periodic_odd_orders(ctx):
    from paper_2308_03140_amd import torch_api as T
    for n, k in ((1, (2, 1, 1)), (3, (1, 2, 2)), (11, (2, 2, 1))):
        _note("direct root, cell of %d" % n)
        c = gen.small_crystal(300 + n, n, kgrid=k)
        args = (torch.tensor(c["coords"], device="cuda"), c["alpha0"] * 0.5, c["omega"], c["rvdw"])
        kw = dict(beta=c["beta"], a=c["a"], lattice=c["lattice"], q_frac=c["q_frac"])
        a = T.evaluate(ctx, *args, eigvals=True, **kw)
        b = T.evaluate(ctx, *args, **kw)
        _same(a, b, 6 * n)
        assert (a["grad_lattice"] - b["grad_lattice"]).abs().max().item() <= 1e-12


def test_workspace_limit(monkeypatch):
    """Limits that the diagonalisation fits and the direct route does not, in
    both orders of use: the calls that were answered under them still are."""
    from paper_2308_03140_amd import torch_api as T
    c = _cluster(91, 100)
    ref_ctx = T.Context(0, "fp64")
    ref = _run(ref_ctx, c)
    n, ld = 300, 320
    mat = 8 * ld * n
    for limit in (3 * mat, 12 * mat, 16 * mat):
        _note("direct root, workspace limit %d" % limit)
        monkeypatch.setenv("MBD_WORKSPACE_LIMIT", str(limit))
        ctx = T.Context(0, "fp64")
        try:
            for rep in range(2):
                e = _run(ctx, c, gradients=False)["energy"].item()
                assert abs(e - ref["energy"].item()) <= 1e-12
                if limit > 3 * mat:
                    a = _run(ctx, c, eigvals=True)
                    _same(a, _run(ctx, c), n)
                    _same(a, ref, n)
        finally:
            ctx.close()
    ref_ctx.close()


def test_decoupled_blocks_fp32_eigenvalues():
    """An FP32 reduction whose columns are at rounding noise of exactly
    decoupled blocks (1e-20, the square below the normal range)."""
    from paper_2308_03140_amd import torch_api as T
    _note("eigh, decoupled blocks with 1e-20 noise")
    ctx = T.Context(0, "fp32_refined")
    try:
        for n in (3, 40, 150):
            rng = np.random.default_rng(n)
            A = rng.standard_normal((n, n))
            A = A + A.T
            M = np.block([[A, np.zeros((n, n))], [np.zeros((n, n)), A]])
            N = rng.standard_normal((2 * n, 2 * n)) * 1e-20
            M += N + N.T
            w, _ = T.eigh(ctx, torch.tensor(M, dtype=torch.float32, device="cuda"))
            assert np.abs(w.double().cpu().numpy() - np.linalg.eigvalsh(M)).max() <= 4e-7 * n ** 0.5 * np.abs(M).sum(1).max()
    finally:
        ctx.close()
