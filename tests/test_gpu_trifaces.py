"""The face kernel of the trilinear apply (a wave per axis over 64 / (2 n)
faces) and the volume kernel that joins its rows: element counts that leave the
last wave of faces and the last block ragged, boundary layers on every axis,
elements that are their own neighbours, reaction, vectors that are not aligned
to two values, and the solvers whose vectors share memory with the face rows.

Tolerances: FP64 1e-12, FP32 / BF16 2e-5 (the bars of the other applies)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1911_01492_amd import inputs as I  # noqa: E402
from paper_1911_01492_amd.dg import DG_OK, DGOperator  # noqa: E402
from tests.gpu_util import banner, bf16_dev, dev, host, rel_l2  # noqa: E402
from tests.test_gpu_trilinear import BCS, box_vertices  # noqa: E402


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("shape,bc", [((7, 3, 2), "dirichlet"), ((5, 2, 4), "periodic"), ((1, 9, 2), "periodic"),
                                      ((1, 1, 3), "dirichlet")])
def test_apply_all_precisions(shape, bc, k):
    banner(f"trilinear faces {shape} {bc} k={k}")
    E = int(np.prod(shape))
    theta, c, V = I.theta(E, seed=k), I.reaction(E), box_vertices(*shape, seed=k)
    m = O.Mesh(*shape, k, bc=BCS[bc], theta=theta, reaction=c, vertices=V)
    op = DGOperator(*shape, k, bc, theta=dev(theta), vertices=dev(V))
    op.set_reaction(dev(c))
    A = O.assemble(m)
    x = I.uniform_vector(m.ndof, seed=k)
    bits = I.to_bf16_bits(x)
    for prec, X, xr, tol in (("f64", dev(x), x, 1e-12),
                             ("f32", dev(I.to_f32(x), torch.float32), I.to_f32(x).astype(np.float64), 2e-5),
                             ("bf16", bf16_dev(bits), I.bf16_bits_to_f64(bits), 2e-5)):
        Y = op.apply(X, prec=prec)
        assert rel_l2(host(Y), A @ xr) <= tol, prec
        buf = torch.empty(m.ndof + 1, dtype=X.dtype, device="cuda")
        buf[1:] = X
        assert torch.equal(op.apply(buf[1:], prec=prec), Y), prec


@pytest.mark.parametrize("k", [1, 3, 7])
def test_solvers_next_to_the_face_rows(k):
    """Solves to 1e-10 (residual checked by the oracle's matrix), an apply between them."""
    shape = (3, 4, 2)
    banner(f"trilinear solvers k={k}")
    V, theta = box_vertices(*shape, seed=3), I.theta(24, seed=2)
    m = O.Mesh(*shape, k, bc=O.DIRICHLET, theta=theta, vertices=V)
    op = DGOperator(*shape, k, "dirichlet", theta=dev(theta), vertices=dev(V))
    A = O.assemble(m)
    bs = I.uniform_vector(m.ndof, seed=9)
    b = dev(bs)
    y = op.apply(b)
    for prec, mode, var in (("f64", "restart", "standard"), ("f64", "restart", "single_reduction"),
                            ("f32", "keep", "standard"), ("bf16", "keep", "standard"), ("f32", "restart", "standard")):
        u, info = op.cg_solve(b, prec_inner=prec, rtol=1e-10, dc_mode=mode, variant=var)
        assert info["status"] == DG_OK, (prec, mode, var)
        assert np.linalg.norm(bs - A @ host(u)) <= 1.2e-10 * np.linalg.norm(bs), (prec, mode, var)
        assert torch.equal(op.apply(b), y)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("shape,bc", [((7, 3, 2), "dirichlet"), ((5, 1, 4), "periodic")])
def test_sensitivity_and_diagonal(shape, bc, k):
    """dA/dtheta (1e-12) from one value per face and the diagonal (1e-13), every degree."""
    banner(f"trilinear dA/dtheta, diagonal {shape} {bc} k={k}")
    E = int(np.prod(shape))
    theta, V = I.theta(E, seed=k), box_vertices(*shape, seed=k)
    m = O.Mesh(*shape, k, bc=BCS[bc], theta=theta, vertices=V)
    op = DGOperator(*shape, k, bc, theta=dev(theta), vertices=dev(V))
    u, v = I.uniform_vector(m.ndof, seed=k), I.uniform_vector(m.ndof, seed=k + 20)
    assert rel_l2(host(op.dA_dtheta(dev(u), dev(v))), O.dA_dtheta(m, u, v)) <= 1e-12
    assert rel_l2(host(op.diagonal()), O.assemble(m).diagonal()) <= 1e-13
