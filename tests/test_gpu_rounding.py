"""How far FP64 results of the direct root are from those of the diagonalisation
(eigvals=True) on the same inputs, at rounding level: residue products from the
order from which they are taken (2470) on, and FP64 products below.

Tolerance: 2-norms of the difference over the result.  Gradients by
diagonalisation are 7e-15 from 64-bit ones (orders 900 to 6000), by FP64 products
likewise: 1e-14 between the two; 1.4 times that is accepted."""
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


@pytest.mark.parametrize("N", [300, 800, 823, 824, 900, 1100])
def test_gradients(ctx, N):
    from paper_2308_03140_amd import torch_api as T
    print("rounding of gradients, N=%d" % N, flush=True)
    c = gen.finite_cluster(8100 + N, N, (N / 0.1) ** (1.0 / 3.0))  # liquid density
    a = (torch.tensor(c["coords"], device="cuda"), 0.5 * c["alpha0"], c["omega"], c["rvdw"])
    x = T.evaluate(ctx, *a, beta=c["beta"], a=c["a"], eigvals=True)
    y = T.evaluate(ctx, *a, beta=c["beta"], a=c["a"])
    for k in ("grad_coords", "grad_rvdw", "grad_alpha0"):
        err = ((x[k] - y[k]).norm() / x[k].norm()).item()
        print("  %s %.1e" % (k, err), flush=True)
        assert err <= 1.4e-14, (k, err)
