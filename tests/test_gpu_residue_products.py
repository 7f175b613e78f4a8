"""Products of the direct root by residues on the INT8 matrix cores (large
orders) against the diagonalisation (eigvals=True) on the same inputs: orders
at the edge of the rule and of the 256-row tiles and 128-column steps, both
precisions, a scratch limit that leaves no room for the residues, and a batch.

Tolerances: those of test_gpu_direct_root for FP64 (both routes carry eps
sqrt(n) times the conditioning of the root); with 12 moduli the operands are
rounded to 2^-47 of their norm, 64 times coarser than FP64."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("energy", "grad_coords", "grad_alpha0", "grad_omega", "grad_rvdw")


def _cluster(seed, N):
    return gen.finite_cluster(seed, N, 12.0 * (N / 32.0) ** (1.0 / 3.0))


def _args(c):
    return (torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"])


def _same(a, b, n, rounding):
    tol = rounding * max(8.0, n ** 0.5) * 30.0 * 4.0
    for k in [k for k in KEYS if k in b]:
        scale = 0.5 * n if k == "energy" else max(1.0 if k == "grad_omega" else 1e-3, a[k].abs().max().item())
        err = (a[k] - b[k]).abs().max().item()
        assert err <= tol * scale, (k, err, tol * scale)


@pytest.mark.parametrize("precision,N", [("fp64", 933), ("fp64", 934), ("fp64", 938), ("fp64", 939), ("fp64", 982),
                                         ("fp32_refined", 799), ("fp32_refined", 800), ("fp32_refined", 853),
                                         ("fp32_refined", 854)])
def test_orders(precision, N):
    from paper_2308_03140_amd import torch_api as T
    print("residue products %s N=%d" % (precision, N), flush=True)
    c = _cluster(2300 + N, N)
    ref = T.Context(0, "fp64")
    ctx = T.Context(0, precision)
    try:
        a = T.evaluate(ref, *_args(c), beta=c["beta"], a=c["a"], eigvals=True)
        b = T.evaluate(ctx, *_args(c), beta=c["beta"], a=c["a"])
        _same(a, b, 3 * N, 2.2e-16 if precision == "fp64" else 64 * 2.2e-16)
        assert abs(a["errors"][0].item() - b["errors"][0].item()) <= 1e-9
    finally:
        ref.close()
        ctx.close()


def test_no_room_for_residues(monkeypatch):
    """The same results where the scratch limit holds the FP64 products only."""
    from paper_2308_03140_amd import torch_api as T
    N = 940
    c = _cluster(2900, N)
    mat = 8 * 2880 * 2820
    print("residue products, scratch limit", flush=True)
    out = []
    for limit in (10 * mat, 40 * mat):
        monkeypatch.setenv("MBD_WORKSPACE_LIMIT", str(limit))
        ctx = T.Context(0, "fp64")
        try:
            out.append(T.evaluate(ctx, *_args(c), beta=c["beta"], a=c["a"]))
        finally:
            ctx.close()
    _same(out[0], out[1], 3 * N, 2.2e-16)


def test_batch():
    from paper_2308_03140_amd import torch_api as T
    print("residue products, batch", flush=True)
    cs = [_cluster(2950 + N, N) for N in (934, 1000)]
    ctx = T.Context(0, "fp64")
    try:
        for _ in range(3):  # eager, captured, replayed
            outs = T.evaluate_batch(ctx, [dict(c, coords=torch.tensor(c["coords"], device="cuda")) for c in cs])
            for c, o in zip(cs, outs):
                assert o["status"] == 0
                a = T.evaluate(ctx, *_args(c), beta=c["beta"], a=c["a"], eigvals=True)
                _same(a, o, 3 * len(c["omega"]), 2.2e-16)
    finally:
        ctx.close()
