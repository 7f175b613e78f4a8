"""Pairwise energy of finite systems at the edges of a row's two wavefronts
(127 to 129 and 256/257 atoms), without damping (s_R = 0), and with a pair so
far apart that it adds nothing, and of cells at the edges of a workgroup's four
pairs, against the oracle; a coincident pair in the last lanes of a row is still
refused.  Bounds of the pairwise path: 1e-11 Ha
per atom, 1e-9 for gradients."""
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


def _run(ctx, c, sR):
    from paper_2308_03140_amd import torch_api as T
    return T.ts_evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"], sR, 20.0)


@pytest.mark.parametrize("N,sR,far", [(127, 0.94, False), (128, 0.94, False), (129, 0.0, False), (256, 0.94, True),
                                      (257, 0.94, False), (3, 0.0, True)])
def test_rows(ctx, N, sR, far):
    print("ts rows N=%d sR=%g far=%d" % (N, sR, far), flush=True)
    c = gen.finite_cluster(1300 + N, N, 12.0 * (N / 32.0) ** (1 / 3))
    if far:
        c["coords"][-1] += 1e9
    ref = oracle.ts(c["coords"], c["alpha0"], c["omega"], c["rvdw"], sR=sR, a=20.0)
    out = _run(ctx, c, sR)
    assert abs(out["energy"].item() - ref["energy"]) / N <= 1e-11
    for k, o in (("grad_R", "grad_coords"), ("grad_alpha0", "grad_alpha0"), ("grad_omega", "grad_omega"),
                 ("grad_rvdw", "grad_rvdw")):
        assert np.abs(out[o].cpu().numpy().reshape(ref[k].shape) - ref[k]).max() <= 1e-9, k


def test_coincident_pair_refused(ctx):
    from paper_2308_03140_amd import torch_api as T
    c = gen.finite_cluster(1400, 200, 24.0)
    c["coords"][199] = c["coords"][3]
    with pytest.raises(T.MBDError) as e:
        _run(ctx, c, 0.94)
    assert e.value.code == 1


@pytest.mark.parametrize("N", [1, 3, 4, 5, 17])
def test_cells(ctx, N):
    from paper_2308_03140_amd import torch_api as T
    print("ts cell N=%d" % N, flush=True)
    c = gen.small_crystal(1500 + N, N)
    ref = oracle.ts(c["coords"], c["alpha0"], c["omega"], c["rvdw"], sR=0.94, a=20.0, lattice=c["lattice"])
    out = T.ts_evaluate(ctx, torch.tensor(c["coords"], device="cuda"), c["alpha0"], c["omega"], c["rvdw"], 0.94, 20.0,
                        lattice=c["lattice"])
    assert abs(out["energy"].item() - ref["energy"]) / N <= 1e-11
    for k, o in (("grad_R", "grad_coords"), ("grad_alpha0", "grad_alpha0"), ("grad_omega", "grad_omega"),
                 ("grad_rvdw", "grad_rvdw")):
        assert np.abs(out[o].cpu().numpy().reshape(ref[k].shape) - ref[k]).max() <= 1e-9, k
