"""The checks of a material field and of coordinates, past the first slice of
their workgroups."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import fem as F
from paper_2602_12365_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda", torch.float64)


@pytest.fixture(scope="module")
def mesh():
    """540,800 triangles and 814,323 coordinates: both past the 512 workgroups of
    1,024 entries that one sweep of the check covers."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(I.TRI3, 520)
    assert m.n_elems > 512 * 1024 and 3 * m.n_nodes > 512 * 1024
    u = 1e-4 * np.random.default_rng(1).standard_normal((m.n_nodes, 3)) * np.array([1.0, 1.0, 0.0])
    op = Operator(I.TRI3, m.X, m.conn)
    yield m, u, op
    op.close()


@pytest.mark.parametrize("at", [512 * 1024 - 1, 512 * 1024, 512 * 1024 + 1024, 540799])
def test_one_element_past_the_first_sweep(mesh, at):
    """One element that differs makes the field varying: the energy changes by a
    millionth, and agrees with the oracle to the energy's 1e-12."""
    m, u, op = mesh
    mu, lam = np.full(m.n_elems, 1.25), np.full(m.n_elems, 2.0)
    op.set_material(dev(mu), dev(lam))
    flat = float(op.energy(dev(u)))
    mu[at] += 0.7
    op.set_material(dev(mu), dev(lam))
    ref = F.FEM(I.TRI3, m.X, m.conn, mu, lam).energy(u)
    assert abs(float(op.energy(dev(u))) - ref) <= 1e-12 * abs(ref)
    assert abs(flat - ref) > 1e-9 * abs(ref)


@pytest.mark.parametrize("at", [512 * 1024 // 3 * 3, 512 * 1024 // 3 * 3 + 3 * 1024, 814323 - 3])
def test_one_coordinate_past_the_first_sweep(mesh, at):
    """One x coordinate moved is noticed (the operator's coordinates change), and
    the energy is the oracle's on the moved mesh to 1e-12."""
    from paper_2602_12365_amd import operator as ops
    m, u, op = mesh
    mu = np.full(m.n_elems, 1.25)
    X = m.X.copy()
    X.reshape(-1)[at] += 0.1 / 520
    psi = float(ops.energy(op, dev(u), dev(mu), dev(2.0 * mu), dev(X)))
    assert torch.equal(op.X, dev(X))
    ref = F.FEM(I.TRI3, X, m.conn, mu, 2.0 * mu).energy(u)
    assert abs(psi - ref) <= 1e-12 * abs(ref)
    ops.energy(op, dev(u), dev(mu), dev(2.0 * mu), dev(m.X))
    assert torch.equal(op.X, dev(m.X))
