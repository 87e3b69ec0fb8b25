"""FP32 and BF16-input applies on affine meshes for every degree (the staged
element tile at n = 3..7 and the constant 1D tables from n = 3 on), on meshes
that leave bricks partly empty and on periodic meshes one element wide, against
the oracle's CSR operator on the rounded input.

Tolerance: the arithmetic error of an FP32 apply is a few hundred units
roundoff (6e-8) at most -- contractions of up to 3 n = 24 terms whose table
entries exceed the result by the ratio of stiffness to residual; 2e-5 is the
bar of the other low-precision tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1911_01492_amd import inputs as I  # noqa: E402
from paper_1911_01492_amd.dg import DGOperator  # noqa: E402
from tests.gpu_util import banner, bf16_dev, dev, host, rel_l2  # noqa: E402

BCS = {"dirichlet": O.DIRICHLET, "periodic": O.PERIODIC}


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("shape,bc", [((3, 2, 2), "dirichlet"), ((1, 3, 2), "periodic")])
def test_f32_and_bf16(shape, bc, k):
    banner(f"low precision {shape} {bc} k={k}")
    E = int(np.prod(shape))
    theta, c = I.theta(E, seed=k), I.reaction(E)
    m = O.Mesh(*shape, k, bc=BCS[bc], theta=theta, reaction=c)
    A = O.assemble(m)
    op = DGOperator(*shape, k, bc, theta=dev(theta))
    op.set_reaction(dev(c))
    x = I.uniform_vector(m.ndof, seed=k)
    x32 = I.to_f32(x)
    bits = I.to_bf16_bits(x)
    for tr in (False, True):
        y = host(op.apply(dev(x32, torch.float32), prec="f32", transpose=tr))
        assert rel_l2(y, A @ x32.astype(np.float64)) <= 2e-5, tr
        y = host(op.apply(bf16_dev(bits), prec="bf16", transpose=tr))
        assert rel_l2(y, A @ I.bf16_bits_to_f64(bits)) <= 2e-5, tr
    Y = host(op.apply_multi(torch.stack([dev(x32, torch.float32), dev(-2 * x32, torch.float32)]), prec="f32"))
    r = A @ x32.astype(np.float64)
    assert rel_l2(Y.reshape(2, -1), np.stack([r, -2 * r])) <= 2e-5


@pytest.mark.parametrize("k", [5, 6, 7])
@pytest.mark.parametrize("shape,bc", [((3, 2, 2), "dirichlet"), ((1, 3, 2), "periodic")])
def test_parallelepipeds_with_constant_tables(shape, bc, k):
    """Equal parallelepipeds in FP32, whose tables are constants from n = 6 on; the same bar."""
    banner(f"low precision parallelepipeds {shape} {bc} k={k}")
    V = I.uniform_vertices(*shape) @ np.array([[1.0, 0.3, -0.2], [0.1, 0.9, 0.25], [-0.15, 0.2, 1.1]]).T
    theta = I.theta(int(np.prod(shape)), seed=k)
    A = O.assemble(m := O.Mesh(*shape, k, bc=BCS[bc], theta=theta, vertices=V))
    op = DGOperator(*shape, k, bc, theta=dev(theta), vertices=dev(V))
    assert op.kernel == "parallelepiped"
    x = I.uniform_vector(m.ndof, seed=k)
    x32, bits = I.to_f32(x), I.to_bf16_bits(x)
    y = host(op.apply(dev(x32, torch.float32), prec="f32"))
    assert rel_l2(y, A @ x32.astype(np.float64)) <= 2e-5
    y = host(op.apply(bf16_dev(bits), prec="bf16"))
    assert rel_l2(y, A @ I.bf16_bits_to_f64(bits)) <= 2e-5
