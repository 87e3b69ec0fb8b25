"""Trilinear applies on meshes far from unit size.  The 1D scalings come from the
element counts, so with the vertices scaled by s the volume and consistency
terms scale by s and the penalty by s^2; the squares of the face areas go like
s^4, are subnormal in FP32 at edges near 1e-10, zero at 1e-12 (where the penalty
is 1e-10 of the rest) and near the largest number at 3e9.

Tolerances: FP64 1e-12; FP32 / BF16 2e-5 (the bars of the other applies)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1911_01492_amd import inputs as I  # noqa: E402
from paper_1911_01492_amd.dg import DGOperator  # noqa: E402
from tests.gpu_util import banner, bf16_dev, dev, host, rel_l2  # noqa: E402
from tests.test_gpu_trilinear import BCS, box_vertices  # noqa: E402


@pytest.mark.parametrize("scale", [8e9, 1e5, 1e-5, 1.5e-9, 6e-10, 1e-10, 4e-12])
@pytest.mark.parametrize("k", [1, 2, 4, 7])
@pytest.mark.parametrize("bc", ["dirichlet", "periodic"])
def test_scaled_vertices(bc, k, scale):
    shape = (4, 3, 2)
    banner(f"trilinear scale {scale} {bc} k={k}")
    E = int(np.prod(shape))
    theta, V = 0.3 * I.theta(E, seed=k), scale * box_vertices(*shape, seed=k)
    m = O.Mesh(*shape, k, bc=BCS[bc], theta=theta, vertices=V)
    op = DGOperator(*shape, k, bc, theta=dev(theta), vertices=dev(V))
    assert op.kernel == "trilinear"
    A = O.assemble(m)
    x = I.uniform_vector(m.ndof, seed=k)
    bits = I.to_bf16_bits(x)
    for prec, X, xr, tol in (("f64", dev(x), x, 1e-12),
                             ("f32", dev(I.to_f32(x), torch.float32), I.to_f32(x).astype(np.float64), 2e-5),
                             ("bf16", bf16_dev(bits), I.bf16_bits_to_f64(bits), 2e-5)):
        assert rel_l2(host(op.apply(X, prec=prec)), A @ xr) <= tol, prec


@pytest.mark.parametrize("k", [1, 3, 6])
def test_subnormal_determinants(k):
    """Elements 3e-11 x 3e-11 x 5e-17: det J straddles FP32's smallest normal number."""
    shape = (4, 3, 2)
    banner(f"trilinear subnormal det k={k}")
    V = 1e-10 * box_vertices(*shape, seed=k) * np.array([1.0, 1.0, 1e-6])
    m = O.Mesh(*shape, k, vertices=V)
    op = DGOperator(*shape, k, "dirichlet", vertices=dev(V))
    x32 = I.to_f32(I.uniform_vector(m.ndof, seed=k))
    y = op.apply(dev(x32, torch.float32), prec="f32")
    assert rel_l2(host(y), O.assemble(m) @ x32.astype(np.float64)) <= 2e-5


@pytest.mark.parametrize("prec,dtype,scale", [("f32", torch.float32, 1e-11), ("f64", torch.float64, 1e-80)])
def test_areas_whose_squares_vanish_stay_finite(prec, dtype, scale):
    shape, k = (4, 3, 2), 2
    banner(f"trilinear scale {scale} {prec}")
    V = scale * box_vertices(*shape, seed=k)
    op = DGOperator(*shape, k, "dirichlet", vertices=dev(V))
    y = op.apply(dev(I.uniform_vector(op.ndof)).to(dtype), prec=prec)
    assert bool(torch.isfinite(y).all())


def test_graded_mesh():
    """Edges from 1e-10 to 1 along x and y in one mesh: the scaling is each face's own."""
    nx, ny, nz, k = 4, 3, 2, 3
    banner("trilinear graded mesh")
    X = np.r_[0.0, 1e-10, 1e-6, 1e-3, 1.0]
    Y = np.r_[0.0, 2e-10, 1e-4, 1.0]
    V = np.array([[X[i] * (1 + 0.1 * l), Y[j] * (1 + 0.05 * i), 0.5 * l * (1 + 0.1 * X[i])]
                  for l in range(nz + 1) for j in range(ny + 1) for i in range(nx + 1)])
    m = O.Mesh(nx, ny, nz, k, vertices=V)
    op = DGOperator(nx, ny, nz, k, "dirichlet", vertices=dev(V))
    assert op.kernel == "trilinear"
    x32 = I.to_f32(I.uniform_vector(m.ndof))
    y = op.apply(dev(x32, torch.float32), prec="f32")
    assert bool(torch.isfinite(y).all())
    assert rel_l2(host(y), O.assemble(m) @ x32.astype(np.float64)) <= 2e-5
