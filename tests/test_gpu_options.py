"""Default block sizes beside the other options of an operator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_12365_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,threads", [(32, 64), (33, 64), (41, 64), (41, 128), (41, 192), (51, 128), (33, 256)])
def test_hexahedra_in_blocks_of_at_most_the_threads(n, threads):
    """A workgroup of few threads gets no more hexahedra than it has threads; FP64
    actions and residuals within 1e-11 of another block size (sums in another
    order), FP32 2e-5."""
    from paper_2602_12365_amd import Operator
    m = I.hex_mesh(n)
    g = np.random.default_rng(n)
    u, v = (torch.as_tensor(s * g.standard_normal((m.n_nodes, 3))).cuda() for s in (0.01 / n, 1.0))
    mu = torch.as_tensor(np.exp(0.3 * g.standard_normal(m.n_elems))).cuda()
    rel = lambda a, b: float((a - b).abs().max() / b.abs().max())  # noqa: E731
    a, b = Operator(I.HEX8, m.X, m.conn, threads=threads), Operator(I.HEX8, m.X, m.conn, block_elems=300)
    assert a.info()["n_blocks"] >= -(-m.n_elems // threads)
    for op in (a, b):
        op.set_material(mu, 1.5 * mu)
        op.linearize(u, "f64")
    assert rel(a.hvp(v), b.hvp(v)) <= 1e-11
    assert rel(a.residual(u), b.residual(u)) <= 1e-11
    assert abs(float(a.energy(u)) - float(b.energy(u))) <= 1e-12 * abs(float(b.energy(u)))
    for op in (a, b):
        op.linearize(u, "f32")
    assert rel(a.hvp(v.float()), b.hvp(v.float())) <= 2e-5
    a.close()
    b.close()


@pytest.mark.parametrize("n,block", [(40, 128), (41, 192), (42, 192), (48, 256), (52, 192), (53, 128), (60, 128), (64, 256)])
def test_hexahedral_blocks_fall_evenly_on_the_cus(n, block):
    """The default of 256 elements gives way to 192 or 128 where that takes an
    eighth off the fullest CU's wave steps (256 CUs); FP64 actions, residuals and
    energies as in blocks of 300."""
    from paper_2602_12365_amd import Operator
    m = I.hex_mesh(n)
    g = np.random.default_rng(n)
    u, v = (torch.as_tensor(s * g.standard_normal((m.n_nodes, 3))).cuda() for s in (0.01 / n, 1.0))
    mu = torch.as_tensor(np.exp(0.3 * g.standard_normal(m.n_elems))).cuda()
    rel = lambda a, b: float((a - b).abs().max() / b.abs().max())  # noqa: E731
    a, b = Operator(I.HEX8, m.X, m.conn), Operator(I.HEX8, m.X, m.conn, block_elems=300)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert a.info()["n_blocks"] == -(-m.n_elems // block)
    for op in (a, b):
        op.set_material(mu, 1.5 * mu)
        op.linearize(u, "f64")
    assert rel(a.hvp(v), b.hvp(v)) <= 1e-11
    assert rel(a.residual(u), b.residual(u)) <= 1e-11
    assert abs(float(a.energy(u)) - float(b.energy(u))) <= 1e-12 * abs(float(b.energy(u)))
    a.close()
    b.close()
