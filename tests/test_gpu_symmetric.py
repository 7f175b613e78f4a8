"""Symmetric systems of identical atoms, alone, in batches and as cells: the
direct root against the diagonalisation (eigvals=True).  Their matrices split
into symmetry sectors that the kernels keep to the last bit, so a start or check
vector of the direct root that is orthogonal to one never sees it: pairs,
chains, squares, rings and grids along the axes and off them, pairs just short
of the collapse and just past it.

Tolerance: eps max(8, sqrt(n)) times the conditioning of the root, times four,
relative to the size of the quantity (dE/domega is a difference of terms near
3/2); lambda_min by the same, relative to itself."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

AXES = {"x": (1, 0, 0), "y": (0, 1, 0), "z": (0, 0, 1), "xz": (2 ** -0.5, 0, -(2 ** -0.5)), "xyz": (3 ** -0.5,) * 3}
KEYS = ("energy", "grad_coords", "grad_alpha0", "grad_omega", "grad_rvdw")


def _system(X, alpha0, beta=0.83):
    n = len(X)
    return {"coords": np.array(X, float), "alpha0": np.full(n, float(alpha0)), "omega": np.full(n, 0.5),
            "rvdw": np.full(n, 3.5), "beta": beta, "a": 6.0}


def _ring(n, r):
    t = 2 * np.pi * np.arange(n) / n
    return np.stack([r * np.cos(t), r * np.sin(t), 0 * t], axis=1)


def _grid(a, b, c, h):
    return h * np.array([[i, j, k] for i in range(a) for j in range(b) for k in range(c)], float)


def _bare(axis, ratio):
    """A pair without damping, 2 alpha0 / r^3 = ratio: collapsed from 1 on."""
    return _system([np.zeros(3), 8.0 * np.array(AXES[axis])], ratio * 8.0 ** 3 / 2, beta=0.0)


def _systems():
    s = {}
    for k, v in AXES.items():
        for al in (25, 40, 50, 60, 80):
            s["pair %s %d" % (k, al)] = _system([np.zeros(3), 7.5 * np.array(v)], al)
        for ratio in (0.9, 0.99, 0.999, 1.01, 1.04):
            s["bare pair %s %g" % (k, ratio)] = _bare(k, ratio)
        for n in (4, 25):
            s["chain %s %d" % (k, n)] = _system([7.5 * i * np.array(v) for i in range(n)], 40)
    for al in (40, 60):
        s["square %d" % al] = _system(_grid(2, 2, 1, 7.5), al)
        s["ring 6 %d" % al] = _system(_ring(6, 7.5), al)
        s["ring 50 %d" % al] = _system(_ring(50, 60.0), al)
    for a, b, c in ((2, 2, 2), (3, 3, 3), (4, 4, 4), (7, 7, 1), (5, 5, 5)):
        s["grid %d %d %d" % (a, b, c)] = _system(_grid(a, b, c, 7.5), 30)
    return s


SYSTEMS = _systems()


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


def _eval(ctx, c, **kw):
    """Outputs, or the status of a collapsed system."""
    from paper_2308_03140_amd import torch_api as T
    try:
        return T.evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"],
                          beta=c["beta"], a=c["a"], **kw)
    except T.CollapseError as e:
        return e.code


def _same(ref, out, tag):
    assert isinstance(ref, int) == isinstance(out, int), (tag, ref, out)
    if isinstance(ref, int):
        assert ref == out
        return
    w = ref["eigvals"].flatten()
    n, kappa = w.numel(), (w.max() / w.min()).item()
    tol = 4 * 2.2e-16 * max(8.0, n ** 0.5) * max(30.0, kappa)
    for k in [k for k in KEYS + ("grad_lattice",) if k in out]:
        size = 0.5 * n if k == "energy" else max(1.0 if k == "grad_omega" else 1e-3, ref[k].abs().max().item())
        err = (ref[k] - out[k]).abs().max().item()
        assert err <= tol * size, (tag, k, err, tol * size)
    low = w.min().item()
    assert abs(out["errors"][0].item() - low) <= tol * low, (tag, out["errors"][0].item(), low)


@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_alone(ctx, name):
    print("symmetric system, %s" % name, flush=True)
    c = SYSTEMS[name]
    ref, out = _eval(ctx, c, eigvals=True), _eval(ctx, c)
    if name.startswith("bare"):
        assert isinstance(ref, int) == (float(name.split()[-1]) > 1.0)
    _same(ref, out, name)
    e = _eval(ctx, c, gradients=False, errors=False)
    assert isinstance(e, int) == isinstance(ref, int)
    if not isinstance(ref, int):
        assert (e["energy"] - out["energy"]).abs().item() <= 1e-12 * len(c["omega"])


@pytest.mark.parametrize("others", [(), (70,), (23, 70, 130)])
def test_batch(ctx, others):
    """All of them in one batch, with members that take the launches of larger
    orders; eager, captured and replayed."""
    from paper_2308_03140_amd import torch_api as T
    print("symmetric systems in a batch, others %s" % (others,), flush=True)
    names = sorted(SYSTEMS)
    mols = [SYSTEMS[k] for k in names] + [gen.finite_cluster(5200 + N, N, 12.0 * (N / 32.0) ** (1 / 3)) for N in others]
    ref = [_eval(ctx, m, eigvals=True) for m in mols]
    for _ in range(3):
        outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
        for i, (r, o) in enumerate(zip(ref, outs)):
            tag = names[i] if i < len(names) else "cluster"
            if isinstance(r, int):
                assert o["status"] == r, tag
            else:
                assert o["status"] == 0, tag
                _same(r, {k: v for k, v in o.items() if k != "status"}, tag)


@pytest.mark.parametrize("cells,kgrid", [((1, 1, 1), (3, 2, 1)), ((1, 1, 1), (4, 4, 2)), ((2, 1, 1), (2, 3, 1)),
                                         ((2, 2, 2), (2, 1, 1)), ((3, 3, 3), (1, 2, 1))])
def test_cubic_cells(ctx, cells, kgrid):
    print("symmetric cell %s, mesh %s" % (cells, kgrid), flush=True)
    for alpha0 in (15.0, 30.0):
        c = _system(_grid(*cells, 8.0), alpha0)
        kw = dict(lattice=np.diag([8.0 * x for x in cells]), kgrid=kgrid)
        _same(_eval(ctx, c, eigvals=True, **kw), _eval(ctx, c, **kw), (cells, kgrid, alpha0))
