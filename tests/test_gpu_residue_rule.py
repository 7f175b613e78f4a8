"""Residue products near the order from which they are taken (2200, both
precisions): its two sides, the last order of a 256-row tile and the first of the
next, against the diagonalisation.

Tolerances as in test_gpu_residue_products: eps sqrt(n) times the conditioning
of the root, with 12 moduli 64 times that (operands rounded to 2^-47 of their
norm); lambda_min by the same rounding, relative to lambda_max."""
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("energy", "grad_coords", "grad_alpha0", "grad_omega", "grad_rvdw")


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("N", [733, 734, 768, 769])
def test_rule(precision, N):
    from paper_2308_03140_amd import torch_api as T
    print("residue rule %s N=%d" % (precision, N), flush=True)
    c = gen.finite_cluster(2600 + N, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))
    a = (torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"])
    ref, ctx = T.Context(0, "fp64"), T.Context(0, precision)
    try:
        x = T.evaluate(ref, *a, beta=c["beta"], a=c["a"], eigvals=True)
        y = T.evaluate(ctx, *a, beta=c["beta"], a=c["a"])
        n = 3 * N
        tol = (1 if precision == "fp64" else 64) * 2.2e-16 * n ** 0.5 * 30.0 * 4.0
        for k in KEYS:
            scale = 0.5 * n if k == "energy" else max(1.0 if k == "grad_omega" else 1e-3, x[k].abs().max().item())
            err = (x[k] - y[k]).abs().max().item()
            assert err <= tol * scale, (k, err, tol * scale)
        w = x["eigvals"][0]
        assert abs(y["errors"][0].item() - w.min().item()) <= tol * w.max().item()
    finally:
        ref.close()
        ctx.close()
