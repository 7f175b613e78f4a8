"""Periodic pair kernels over the ways their lanes are dealt out: q counts that
leave one lane per pair or more than one group of q points, few pairs (whose
images are then split over the lanes of a wavefront or of a workgroup) and
many, against the oracle.  FP64 sums in another order than the oracle's: the
energy and every gradient agree to rounding, about 1e-13 of sums of order 1."""
import sys

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2308_03140_amd import torch_api as T
    c = T.Context(0, "fp64")
    yield c
    c.close()


@pytest.mark.parametrize("N,nq", [(1, 1), (2, 1), (5, 1), (7, 3), (16, 1), (20, 5), (4, 65), (30, 2), (6, 33)])
def test_pair_layouts(ctx, N, nq):
    from paper_2308_03140_amd import torch_api as T
    _note("periodic pairs N=%d nq=%d" % (N, nq))
    c = gen.small_crystal(500 + N, N, kgrid=(1, 1, 1), side_scale=max(0.6, (N / 64.0) ** (1.0 / 3.0)))
    q = np.random.default_rng(N * 100 + nq).uniform(-0.5, 0.5, (nq, 3))
    # half polarisabilities and wide radii keep the dense cells outside the collapse
    args = (c["alpha0"] * 0.3, c["omega"], c["rvdw"])
    ref = oracle.mbd_periodic(c["coords"], c["lattice"], q, *args, c["beta"], c["a"])
    out = T.evaluate(ctx, torch.tensor(c["coords"], device="cuda"), *args, beta=c["beta"], a=c["a"],
                     lattice=c["lattice"], q_frac=q)
    assert abs(out["energy"].item() - ref["energy"]) <= 1e-12 * N
    for k, o in (("grad_R", "grad_coords"), ("grad_alpha0", "grad_alpha0"), ("grad_omega", "grad_omega"),
                 ("grad_rvdw", "grad_rvdw"), ("grad_lattice", "grad_lattice")):
        err = np.abs(out[o].cpu().numpy().reshape(np.shape(ref[k])) - ref[k]).max()
        assert err <= 1e-11, (k, err)
