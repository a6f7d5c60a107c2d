"""Invariances that hold in FP64 (and FP32) arithmetic, not only on paper: the
operators see differences of nodal values within an element, so a constant
added to the coordinates, the displacement or the direction changes nothing
beyond the order of the nodal sums.  The values are dyadic with few bits, so
that the constant is added without rounding and every difference is the same
number with and without it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_12365_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda", dtype=dtype)


def dyadic(a, bits):
    return np.round(np.asarray(a) * 2.0 ** bits) / 2.0 ** bits


def rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


def passes(op, u, v, model):
    """Every pass that reads coordinates and displacement apart."""
    out = {"residual": op.residual(u), "diag": op.jacobi_diag(u)}
    if model != "transport":
        out["energy"] = op.energy(u).clone()
        out["offdiag"] = op.jacobi_offdiag(u)
        out["dmu"], out["dlam"] = op.grad_material(u)
        out["vmu"], out["vlam"] = op.residual_vjp_material(u, v)
        out["dX"] = op.grad_coords(u)
    return out


@pytest.mark.parametrize("what", ["coordinates", "displacement", "direction"])
@pytest.mark.parametrize("model", ["neo_hookean", "linear", "transport"])
@pytest.mark.parametrize("elem,n", [(I.HEX8, 5), (I.HEX8, 8), (I.TET4, 4), (I.TRI3, 6)])
def test_a_constant_added_changes_nothing(elem, n, model, what):
    """Values of an element are computed from the same differences, so per-element
    results and the energy agree to 1e-15 (the energy's sum order is fixed); nodal
    sums add at most 8 elements' shares of a few times the largest sum in any
    order, 8 * 2^-53 * 10: 1e-14, FP32 shares summed in FP64 the same and the
    result's rounding, 2^-23.  Transport without velocity and reaction sees the
    differences alone as well."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(elem, n)
    g = np.random.default_rng(n)
    planar = np.array([1.0, 1.0, 0.0]) if elem == I.TRI3 else np.ones(3)
    X = dyadic(m.X + 0.1 / n * g.standard_normal(m.X.shape) * planar, 20)
    u, v = dyadic(0.02 / n * g.standard_normal(X.shape) * planar, 24), dyadic(g.standard_normal(X.shape) * planar, 8)
    mu = dev(np.exp(0.3 * g.standard_normal(m.n_elems)))
    lam = 1.5 * mu if model != "transport" else 0.0 * mu
    shift = 2.0 ** 14 * planar

    def operator(X):
        op = Operator(elem, X, m.conn, model=model)
        op.set_material(mu, lam)
        return op

    op = operator(X)
    if what == "direction":
        for prec, dtype, tol in (("f64", torch.float64, 1e-14), ("f32", torch.float32, 1e-14 + 2.0 ** -23)):
            op.linearize(dev(u), prec)
            assert rel(op.hvp(dev(v + shift, dtype)), op.hvp(dev(v, dtype))) <= tol
    else:
        want = passes(op, dev(u), dev(v), model)
        moved = operator(X + shift) if what == "coordinates" else op
        got = passes(moved, dev(u + shift if what == "displacement" else u), dev(v), model)
        for k in want:
            tol = 1e-15 if k in ("energy", "dmu", "dlam", "vmu", "vlam") else 1e-14
            assert rel(got[k], want[k]) <= tol, k
        if moved is not op:
            moved.close()
    op.close()
