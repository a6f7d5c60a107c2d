"""Edges of the launch rules: sizes at which a kernel's tiles, remainders or
choice of path change, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import fem as F
from paper_2602_12365_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(a, dtype=None):
    t = torch.as_tensor(a)
    return t.to("cuda", dtype if dtype is not None else t.dtype)


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("at", [0, 1, 255, 1023, 1024, 1295])
def test_uniform_check_finds_one_element(at):
    """One element that differs, anywhere in the check's slices of 1024, makes
    the field varying; a uniform field afterwards is uniform again (energies
    within the energy's 1e-12 of the oracle)."""
    from paper_2602_12365_amd import Operator
    m = I.tet_mesh(6)
    u = I.gaussian_field(m.n_nodes, 0.01, 3)
    op = Operator(I.TET4, m.X, m.conn)
    for bump_mu, bump_lam in ((0.7, 0.0), (0.0, 0.0), (0.0, -0.4), (0.0, 0.0)):
        mu, lam = np.full(m.n_elems, 1.25), np.full(m.n_elems, 2.0)
        mu[at] += bump_mu
        lam[at] += bump_lam
        op.set_material(dev(mu), dev(lam))
        ref = F.FEM(I.TET4, m.X, m.conn, mu, lam).energy(u)
        assert abs(float(op.energy(dev(u))) - ref) <= 1e-12 * abs(ref)
