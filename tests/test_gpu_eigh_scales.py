"""Eigen-decompositions of matrices at the ends of the floating-point range,
subnormal ones among them (their reciprocal norm overflows): results are finite
and as large as the matrix.  Reflectors of columns whose squares leave the range
are left out, so no digits are asked for there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 3, 40, 150, 300])
@pytest.mark.parametrize("exponent", [-1072, -1060, -1024, -1000, -900])
def test_tiny(n, exponent):
    from paper_2308_03140_amd import torch_api as T
    print("eigh of order %d at 2^%d" % (n, exponent), flush=True)
    A = np.random.default_rng(n).standard_normal((2, n, n))
    A = np.ldexp(A + A.transpose(0, 2, 1), exponent)
    ctx = T.Context(0, "fp64")
    try:
        for vectors in (False, True):
            w, Z = T.eigh(ctx, torch.tensor(A, device="cuda"), vectors=vectors)
            w = w.cpu().numpy()
            assert np.isfinite(w).all() and (np.diff(w, axis=1) >= 0).all()
            assert np.abs(w).max() <= n * np.abs(A).max()
            if vectors:
                G = (Z.transpose(1, 2) @ Z).cpu().numpy()
                assert np.abs(G - np.eye(n)).max() <= 1e-12
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [40, 150, 300])
@pytest.mark.parametrize("dtype,exponent", [("float32", -73), ("float32", -68), ("float64", -535), ("float64", -515)])
def test_squares_below_the_normal_range(n, dtype, exponent):
    """Every reflector of such a matrix is left out: refused, not answered with
    the eigenvalues of its diagonal."""
    from paper_2308_03140_amd import torch_api as T
    print("eigh of order %d at 2^%d, %s" % (n, exponent, dtype), flush=True)
    A = np.random.default_rng(n).standard_normal((n, n))
    A = torch.tensor(np.ldexp(A + A.T, exponent), dtype=getattr(torch, dtype), device="cuda")
    ctx = T.Context(0, "fp64")
    try:
        for vectors in (False, True):
            with pytest.raises(T.MBDError) as e:
                T.eigh(ctx, A, vectors=vectors)
            assert e.value.code == 1
    finally:
        ctx.close()
