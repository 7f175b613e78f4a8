"""Which systems of an FP32 + refinement context go through the FP32
eigenvectors: all below the order from which residue products with 12 moduli
pay (2128), every batch with one of them and every cell.  Their error
estimates (errors[1..3]) are those of a call that also asks for eigenvalues,
which is always diagonalised; a system that takes the direct root reports
none."""
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp32_refined")
    yield c
    c.close()


def _cluster(N):
    return gen.finite_cluster(700 + N, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))


def _eval(ctx, c, **kw):
    from paper_2308_03140_amd import torch_api as T
    return T.evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"],
                      beta=c["beta"], a=c["a"], **kw)


def _refined(errors, ref):
    """As many refinement steps as the diagonalised call took, from FP32
    eigenvectors as far from orthogonal as its own (the order of the FP32 sums
    is not fixed)."""
    e, r = errors.tolist(), ref.tolist()
    assert r[2] >= 1.0 and e[2] == r[2], (e, r)
    assert r[1] / 4.0 <= e[1] <= 4.0 * r[1], (e, r)


@pytest.mark.parametrize("N", [2, 21, 43, 150, 301, 701, 709])
def test_below_the_line(ctx, N):
    print("FP32 route N=%d" % N, flush=True)
    c = _cluster(N)
    _refined(_eval(ctx, c)["errors"], _eval(ctx, c, eigvals=True)["errors"])


def test_from_the_line_on(ctx):
    print("FP32 route N=710", flush=True)
    assert _eval(ctx, _cluster(710), gradients=False)["errors"].tolist()[1:] == [0.0, 0.0, 0.0]


def test_batches(ctx):
    from paper_2308_03140_amd import torch_api as T
    for sizes in ((10, 60, 130), (710, 43)):
        print("FP32 route, batch of %s" % (sizes,), flush=True)
        mols = [_cluster(N) for N in sizes]
        ref = [_eval(ctx, m, eigvals=True)["errors"] for m in mols]
        for _ in range(3):  # eager, captured, replayed
            outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
            for o, r in zip(outs, ref):
                assert o["status"] == 0
                _refined(o["errors"], r)


def test_cells(ctx):
    print("FP32 route, cell", flush=True)
    c = gen.small_crystal(311, 11, kgrid=(2, 2, 1))
    c["alpha0"] = c["alpha0"] * 0.5
    kw = dict(lattice=c["lattice"], kgrid=(2, 2, 1))
    _refined(_eval(ctx, c, **kw)["errors"], _eval(ctx, c, eigvals=True, **kw)["errors"])
