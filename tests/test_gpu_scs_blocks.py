"""Screening at the edges of the Cholesky panels and tiles (orders 3 N around
16, 32, 64, 128, 192, 256, 320 and 512) against the oracle: the screened
parameters to the 1e-12 of the screening stage, the forces, whose chain rule
solves with the same factors, to the path's 1e-6."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


@pytest.mark.parametrize("N", [3, 5, 6, 11, 16, 21, 22, 42, 43, 64, 65, 85, 86, 107, 171])
def test_blocks(ctx, N):
    from paper_2308_03140_amd import torch_api as T
    print("scs blocks N=%d" % N, flush=True)
    c = gen.finite_cluster(1600 + N, N, 12.0 * (N / 32.0) ** (1 / 3))
    scs = oracle.scs(c["coords"], c["alpha0"], c["omega"], c["rvdw"], c["beta"], c["a"], nfreq=3)
    ref = oracle.mbd_rsscs(c["coords"], c["alpha0"], c["omega"], c["rvdw"], c["beta"], c["a"], nfreq=3)
    out = T.rsscs_evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"],
                           beta=c["beta"], a=c["a"], n_freq=3)
    p = out["scs"].cpu().numpy()
    for row, k in enumerate(("alpha", "c6", "omega", "rvdw")):
        np.testing.assert_allclose(p[row], scs[k], rtol=1e-12, err_msg=k)
    assert np.abs(out["grad_coords"].cpu().numpy() - ref["grad_R"]).max() <= 1e-6

