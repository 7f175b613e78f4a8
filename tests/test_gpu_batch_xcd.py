"""Batches whose matrices are dealt out to the XCDs whole: counts around the
multiples of eight at which the rule turns, mixed orders (equal ones among
them), each member against its own evaluation; and a cell's q points together
against each of them alone.  Both sides run the same arithmetic on the same
matrix up to the tile shape: 1e-12 relative (energies), 1e-11 of the largest
component (gradients)."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


@pytest.mark.parametrize("count", [2, 7, 8, 9, 14, 15, 16, 17, 64, 65])
def test_batch_members(ctx, count):
    from paper_2308_03140_amd import torch_api as T
    print("xcd batch of %d" % count, flush=True)
    rng = np.random.default_rng(count)
    sizes = [int(x) for x in rng.integers(22, 60, count)]
    sizes[0] = sizes[-1] = 59
    mols = [gen.finite_cluster(4100 + m, N, 12.0 * (N / 32.0) ** (1 / 3)) for m, N in enumerate(sizes)]
    outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
    for m, o in zip(mols, outs):
        one = T.evaluate(ctx, torch.tensor(m["coords"], device="cuda"), m["alpha0"], m["omega"], m["rvdw"],
                         beta=m["beta"], a=m["a"])
        assert o["status"] == 0
        assert abs(o["energy"].item() - one["energy"].item()) <= 1e-12 * len(m["omega"])
        g = one["grad_coords"].abs().max().item()
        assert (o["grad_coords"] - one["grad_coords"]).abs().max().item() <= 1e-11 * max(g, 1e-3)


@pytest.mark.parametrize("nq", [7, 8, 9, 16])
def test_q_points(ctx, nq):
    from paper_2308_03140_amd import torch_api as T
    print("xcd %d q points" % nq, flush=True)
    c = gen.small_crystal(4300, 13)
    rng = np.random.default_rng(nq)
    qf = rng.uniform(-0.45, 0.45, (nq, 3))
    run = lambda q: T.evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"],
                               beta=c["beta"], a=c["a"], lattice=c["lattice"], q_frac=q)
    out = run(qf)
    ones = [run(qf[i:i + 1]) for i in range(nq)]
    assert abs(out["energy"].item() - np.mean([o["energy"].item() for o in ones])) <= 1e-12 * 13
    g = torch.stack([o["grad_coords"] for o in ones]).mean(0)
    assert (out["grad_coords"] - g).abs().max().item() <= 1e-11 * max(g.abs().max().item(), 1e-3)
