"""Small systems in a batch of large ones: their Lanczos recurrences span the
whole space long before the launches that the large ones need end, and their
smallest eigenvalues are still those of their own evaluations with
eigenvalues (1e-12 relative)."""
import pytest

import gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("big", [90, 160])
def test_small_members(big):
    from paper_2308_03140_amd import torch_api as T
    print("small members beside %d atoms" % big, flush=True)
    ctx = T.Context(0, "fp64")
    try:
        mols = [gen.finite_cluster(5200 + N, N, 12.0 * (N / 32.0) ** (1 / 3)) for N in (big, 1, 2, 3, 5, 7, 9, 12, 16)]
        outs = T.evaluate_batch(ctx, [dict(m, coords=torch.tensor(m["coords"], device="cuda")) for m in mols])
        for m, o in zip(mols, outs):
            one = T.evaluate(ctx, torch.tensor(m["coords"], device="cuda"), m["alpha0"], m["omega"], m["rvdw"],
                             beta=m["beta"], a=m["a"], eigvals=True)
            assert o["status"] == 0
            ref = one["eigvals"][0].min().item()
            assert abs(o["errors"][0].item() - ref) <= 1e-12 * ref, (len(m["omega"]), o["errors"][0].item(), ref)
            assert abs(o["energy"].item() - one["energy"].item()) <= 1e-11 * len(m["omega"])
    finally:
        ctx.close()
