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


@pytest.mark.parametrize("rows", [1, 15, 17, 64, 65, 2048 * 16 + 5])
def test_mlp_gradient_at_row_remainders(rows):
    """Loss gradient at the edges of the 16-row steps, the 64-row workgroups
    and the grid's 2048 waves, against the float64 backward pass on the bf16
    activations of the library's own forward (hidden activations are equal to
    the last bit but for roundings at a bfloat16 boundary, so only FP32 sums
    differ: each parameter's gradient within (rows + 130) 2^-24 of its sum of
    absolute terms, rows capped at a wave's 512)."""
    from paper_2602_12365_amd import Operator, _lib as L, precond as PC
    g = np.random.default_rng(rows)
    m = I.hex_mesh(2)
    op = Operator(I.HEX8, m.X, m.conn)
    theta = PC.init_params(3)
    k = L.EFEM_MLP_OUT * (L.EFEM_MLP_HID + 1)
    theta[-k:] += dev(0.2 * g.standard_normal(k), torch.float32)
    x = np.zeros((rows, 16), dtype=np.float32)
    x[:, :12] = g.standard_normal((rows, 12))
    xb = torch.as_tensor(x).bfloat16()
    aux = np.zeros((rows, L.EFEM_MLP_AUX), dtype=np.float32)
    aux[:, :6] = g.standard_normal((rows, 6))
    aux[:, 6:9] = g.random((rows, 3)) > 0.1
    aux[:, 9] = np.exp(0.3 * g.standard_normal(rows))
    aux[:, 10] = 1.0 / rows
    op.set_mlp(theta)
    X = xb.view(torch.int16).cuda()
    h1, h2, out = op.mlp_forward_layers(X)
    grad, loss = op.mlp_loss_grad(X, dev(aux), theta)
    d = lambda t: t.cpu().double().numpy()  # noqa: E731
    h1, h2, out = (d(t.view(torch.bfloat16) if t.dtype == torch.int16 else t) for t in (h1, h2, out))
    t = d(theta.bfloat16())
    W1, b1, W2, b2, W3 = (t[:768].reshape(64, 12), t[768:832], t[832:4928].reshape(64, 64), t[4928:4992],
                          t[4992:5184].reshape(3, 64))
    xd, ad = d(xb)[:, :12], aux.astype(np.float64)
    e = ad[:, 6:9] * (ad[:, 0:3] + ad[:, 9:10] * out) - ad[:, 6:9] * ad[:, 3:6]
    do = 2.0 * ad[:, 10:11] * ad[:, 9:10] * ad[:, 6:9] * e
    sig = lambda a: 1.0 / (1.0 + np.exp(-a))  # noqa: E731
    s2, s1 = sig(h1 @ W2.T + b2), sig(xd @ W1.T + b1)
    d2 = (do @ W3) * s2
    d1 = (d2 @ W2) * s1
    parts = ((d1, xd), (d1, None), (d2, h1), (d2, None), (do, h2), (do, None))
    ref = np.concatenate([(a.T @ b if b is not None else a.sum(0)).ravel() for a, b in parts])
    # magnitudes of the terms, cancellation inside the deltas included
    m_do = 2.0 * np.abs(ad[:, 10:11] * ad[:, 9:10] * ad[:, 6:9]) * (
        np.abs(ad[:, 0:3]) + np.abs(ad[:, 9:10]) * (np.abs(h2) @ np.abs(W3).T + 1.0) + np.abs(ad[:, 3:6]))
    m2 = (m_do @ np.abs(W3)) * (s2 + 1e-3)
    m1 = (m2 @ np.abs(W2)) * (s1 + 1e-3)
    mags = ((m1, xd), (m1, None), (m2, h1), (m2, None), (m_do, h2), (m_do, None))
    mag = np.concatenate([(np.abs(a).T @ np.abs(b) if b is not None else a.sum(0)).ravel() for a, b in mags])
    err = np.abs(d(grad) - ref)
    tol = (min(rows, 512) + 130) * 2.0 ** -24 * mag + 1e-30
    assert (err <= tol).all(), (err / tol).max()
    assert abs(float(loss) - (ad[:, 10:11] * e * e).sum()) <= 1e-5 * float(loss)


def _fan(n):
    """n triangles around one hub node (its ring holds n + 1 nodes)."""
    a = 2.0 * np.pi * np.arange(n) / n
    X = np.concatenate([[[0.0, 0.0, 0.0]], np.stack([np.cos(a), np.sin(a), 0.0 * a], axis=1)])
    k = np.arange(n)
    conn = np.stack([0 * k, 1 + k, 1 + (k + 1) % n], axis=1).astype(np.int32)
    return I.Mesh(I.TRI3, n, X, conn)


@pytest.mark.parametrize("model", ["neo_hookean", "linear"])
@pytest.mark.parametrize("mesh", ["fan254", "fan255", "fan300", "tet1", "tet5s", "hex1", "hex5s"])
def test_assembly_by_rows_and_by_colours(mesh, model):
    """Sparse assembly at the rule's line (a ring of 255 nodes goes by rows,
    256 by colours), on one cell and on meshes that leave partly filled waves,
    free and with prescribed DOFs, against the oracle's tangent (1e-10)."""
    from paper_2602_12365_amd import Operator
    if mesh.startswith("fan"):
        m = _fan(int(mesh[3:]))
    else:
        m = I.make_mesh(I.TET4 if mesh[0] == "t" else I.HEX8, int(mesh[3]))
        m = I.scrambled_mesh(m, 5) if mesh.endswith("s") else m
    g = np.random.default_rng(4)
    mu = np.exp(0.3 * g.standard_normal(m.n_elems))
    u = 0.02 / max(m.n, 1) * g.standard_normal((m.n_nodes, 3))
    if mesh.startswith("fan"):
        u = 1e-4 * g.standard_normal((m.n_nodes, 3))
    op = Operator(m.elem, m.X, m.conn, model=model)
    op.set_material(dev(mu), dev(1.5 * mu))
    K = F.FEM(m.elem, m.X, m.conn, mu, 1.5 * mu, model=model).tangent_matrix(u)
    K.sort_indices()
    got = op.sparse_assemble(dev(u)).cpu().numpy()
    assert np.abs(got - K.data).max() <= 1e-10 * np.abs(K.data).max()
    mask = (g.random(3 * m.n_nodes) < 0.3).astype(np.uint8)
    op.set_dirichlet(dev(mask))
    got = op.sparse_assemble(dev(u)).cpu().numpy()
    C = K.tocoo()
    C.data = np.where((mask[C.row] == 0) & (mask[C.col] == 0), C.data, 0.0)
    C = C.tocsr()
    C.sort_indices()
    assert np.abs(got - C.data).max() <= 1e-10 * np.abs(K.data).max()


@pytest.mark.parametrize("model", ["neo_hookean", "linear"])
@pytest.mark.parametrize("n,block", [(1, 0), (2, 3), (3, 0), (3, 17), (4, 63), (5, 0), (5, 65)])
def test_hexahedra_at_lane_remainders(n, block, model):
    """Hex8 passes with blocks that end inside a wave's 16 elements, with a
    varying material (every element finds its own), a mask and the adjoints:
    FP64 1e-10 and FP32 5e-5 of the largest entry."""
    from paper_2602_12365_amd import Operator
    m = I.scrambled_mesh(I.hex_mesh(n), 3) if n > 1 else I.hex_mesh(1)
    g = np.random.default_rng(n)
    mu = np.exp(0.4 * g.standard_normal(m.n_elems))
    lam = np.exp(0.4 * g.standard_normal(m.n_elems))
    u, v = 0.03 / n * g.standard_normal((2, m.n_nodes, 3))
    op = Operator(I.HEX8, m.X, m.conn, model=model, block_elems=block)
    op.set_material(dev(mu), dev(lam))
    orc = F.FEM(I.HEX8, m.X, m.conn, mu, lam, model=model)
    for mask in (None, (g.random(3 * m.n_nodes) < 0.3).astype(np.uint8)):
        op.set_dirichlet(None if mask is None else dev(mask))
        free = np.ones((m.n_nodes, 3)) if mask is None else 1.0 - mask.reshape(-1, 3)
        want = orc.hvp(u, v * free) * free
        op.linearize(dev(u), "f64")
        assert np.abs(op.hvp(dev(v)).cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()
        op.linearize(dev(u), "f32")
        got = op.hvp(dev(v, torch.float32)).cpu().numpy()
        assert np.abs(got - want).max() <= 5e-5 * np.abs(want).max()
        res = orc.residual(u) * free
        assert np.abs(op.residual(dev(u)).cpu().numpy() - res).max() <= 1e-10 * np.abs(res).max()
        d = np.where(free > 0, orc.jacobi_diag(u).reshape(-1, 3), 1.0)
        assert rel(op.jacobi_diag(dev(u)).cpu(), d) <= 1e-10
    op.set_dirichlet(None)
    psi = orc.energy(u)
    assert abs(float(op.energy(dev(u))) - psi) <= 1e-12 * abs(psi)
    assert rel(op.jacobi_offdiag(dev(u)).cpu(), orc.jacobi_offdiag(u).reshape(-1, 3)) <= 1e-10
    for got, want in zip(op.grad_material(dev(u)), orc.grad_material(u)):
        assert rel(got.cpu(), want) <= 1e-10
    for got, want in zip(op.residual_vjp_material(dev(u), dev(v)), orc.residual_vjp_material(u, v)):
        assert rel(got.cpu(), want) <= 1e-10
    assert rel(op.grad_coords(dev(u)).cpu(), orc.grad_coords(u).reshape(-1, 3)) <= 1e-10


@pytest.mark.parametrize("scatter", ["halo", "color", "atomic"])
@pytest.mark.parametrize("elem,n,block", [(I.TET4, 1, 0), (I.TET4, 4, 0), (I.TET4, 4, 40), (I.HEX8, 2, 0),
                                          (I.HEX8, 4, 7), (I.TRI3, 6, 9)])
def test_krylov_iterations_by_scatter(elem, n, block, scatter):
    """PCG whose step sums the shared nodes' halo slots (or reads every node,
    on one block and under the other scatters), with both preconditioners and
    models: the true residual meets the tolerance (rtol 1e-9, and the FP64
    recursion's drift, 1e-10), an FP32 solve its own accuracy (1e-4), b = 0
    gives 0, and a cap of one iteration returns after the first check."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(elem, n)
    m = I.scrambled_mesh(m, 8) if elem != I.TRI3 and n > 1 else m
    g = np.random.default_rng(2)
    mu = np.exp(0.3 * g.standard_normal(m.n_elems))
    mask = I.clamp_planar(m.X, 0.1)[0] if elem == I.TRI3 else (m.X[:, 2:] < 1e-9).repeat(3, 1).astype(np.uint8).ravel()
    free = 1.0 - mask.reshape(-1, 3)
    u = 0.005 / n * g.standard_normal((m.n_nodes, 3)) * free
    b = g.standard_normal((m.n_nodes, 3))
    for model in ("neo_hookean", "linear"):
        op = Operator(elem, m.X, m.conn, scatter=scatter, block_elems=block, model=model)
        op.set_material(dev(mu), dev(1.5 * mu))
        op.set_dirichlet(dev(mask))
        orc = F.FEM(elem, m.X, m.conn, mu, 1.5 * mu, model=model)
        bn = np.linalg.norm(b * free)
        for precond in (0, 2):
            x, it, _ = op.linear_solve(dev(u), dev(b), rtol=1e-9, precond=precond)
            x = x.cpu().numpy()
            assert it > 0 and np.all(x[mask.reshape(-1, 3) == 1] == 0.0)
            assert np.linalg.norm((b - orc.hvp(u, x)) * free) <= (1e-9 + 1e-10) * bn
            x32 = op.linear_solve(dev(u), dev(b), rtol=1e-6, hvp_prec="f32", precond=precond)[0].cpu().numpy()
            assert np.abs(x32 - x).max() <= 1e-4 * np.abs(x).max()
            assert float(op.linear_solve(dev(u), dev(0.0 * b), precond=precond)[0].abs().max()) == 0.0
            assert op.linear_solve(dev(u), dev(b), rtol=1e-9, precond=precond, max_iter=1)[1] <= 8
        op.close()


@pytest.mark.parametrize("elem,n,chunks", [
    (I.TRI3, 19, False), (I.TRI3, 20, False), (I.TRI3, 362, False), (I.TRI3, 363, False), (I.TET4, 3, False),
    (I.TET4, 4, False), (I.TET4, 5, False), (I.TET4, 32, False), (I.TET4, 33, False), (I.TET4, 50, False),
    (I.TET4, 51, True), (I.TET4, 57, True), (I.HEX8, 32, False), (I.HEX8, 33, False)])
def test_default_blocks_by_mesh_size(elem, n, chunks):
    """Default block sizes and the choice of the chunk pass at the edges of
    their rules (722 and 800 triangles, 2^18 and above; tetrahedra below and
    above 384 a block, 512 blocks and two blocks per CU; hexahedra at 512
    blocks of 64), against a caller's blocks of 300: FP64 actions, residuals
    and diagonals within 1e-11 (sums in another order), FP32 2e-5."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(elem, n)
    dim = m.X.shape[1]
    g = np.random.default_rng(n)
    u, v = (dev(s * g.standard_normal((m.n_nodes, dim))) for s in (0.01 / n, 1.0))
    mu = dev(np.exp(0.3 * g.standard_normal(m.n_elems)))
    a, b = (Operator(elem, m.X, m.conn, block_elems=be, chunks=be == 0) for be in (0, 300))
    assert (a.info()["n_chunks"] > 0) == chunks
    for op in (a, b):
        op.set_material(mu, 1.5 * mu)
    for what in (lambda op: op.residual(u), lambda op: op.jacobi_diag(u),
                 lambda op: (op.linearize(u, "f64"), op.hvp(v))[1]):
        assert rel(what(a).cpu(), what(b).cpu()) <= 1e-11
    for op in (a, b):
        op.linearize(u, "f32")
    assert rel(a.hvp(v.float()).cpu(), b.hvp(v.float()).cpu()) <= 2e-5
    assert abs(float(a.energy(u)) - float(b.energy(u))) <= 1e-12 * abs(float(b.energy(u)))
    a.close()
    b.close()


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("mesh", ["tet1", "tet3s", "hex1", "hex3s", "fan9"])
def test_features_at_ragged_rings(mesh, masked):
    """Both kinds of node features in one pass, on 1-rings of 3 to 26 nodes
    (the fan: a hub of 10, rims of 4), whose lengths leave every remainder of
    the pass's four neighbours: within one bfloat16 ulp of the float64 features
    (FP32 sums lie within 1e-6 of them, which can cross one rounding boundary)."""
    from oracle import precond as P
    from paper_2602_12365_amd import Operator, precond as PC
    elem = I.HEX8 if mesh[:3] == "hex" else I.TET4
    if mesh[:3] == "fan":
        k = int(mesh[3:])
        a = 2 * np.pi * np.arange(k) / k
        X = np.concatenate([[[0.0, 0, 0], [0, 0, 1.0]], np.stack([np.cos(a), np.sin(a), 0 * a], 1)])
        conn = np.stack([np.zeros(k), 2 + np.arange(k), 2 + (np.arange(k) + 1) % k, np.ones(k)], 1).astype(np.int32)
    else:
        m = I.make_mesh(elem, int(mesh[3]))
        m = I.scrambled_mesh(m, 4) if mesh.endswith("s") else m
        X, conn = m.X, m.conn
    n = X.shape[0]
    g = np.random.default_rng(n)
    mask = (g.random(3 * n) < (0.3 if masked else 0.0)).astype(np.uint8)
    op = Operator(elem, X, conn)
    op.set_mlp(PC.init_params(1))
    if masked:
        op.set_dirichlet(dev(mask))
    diag = np.exp(g.standard_normal((n, 3)))
    r, t = (g.standard_normal((n, 3)).astype(np.float32) for _ in range(2))
    rows, aux = op.precond_rows(dev(r), dev(diag), dev(t), 1.0)
    ref, gref, sref = P.features(r, diag, mask, *P.node_neighbours(conn, n))
    bits = rows.cpu().numpy().view(np.uint16).astype(np.uint32) << 16
    got = bits.view(np.float32)[:, :12].astype(np.float64)
    assert np.all(np.abs(got - P.bf16_round(ref.astype(np.float32))) <= 2.0 ** -7 * np.abs(ref) + 1e-6)
    a = aux.cpu().numpy()
    assert np.abs(a[:, :3] - gref).max() <= 1e-6 * np.abs(gref).max()
    assert np.allclose(a[:, 9], sref, rtol=1e-5)


@pytest.mark.parametrize("elem,n,block,threads", [
    (I.TET4, 2, 4, 0), (I.TET4, 5, 40, 0), (I.TET4, 5, 40, 64), (I.TET4, 8, 0, 0), (I.HEX8, 6, 0, 0),
    (I.HEX8, 7, 0, 0), (I.TRI3, 12, 18, 0), (I.TRI3, 12, 8, 0), (I.TRI3, 24, 0, 0), (I.TET4, 10, 0, 0)])
def test_last_workgroup_finishes(elem, n, block, threads):
    """Passes of few blocks whose last workgroup gathers the shared nodes and
    sums the energy, and those just past that rule (more shared nodes than
    threads, more blocks): against the colour scatter (1e-11, FP32 2e-5) and
    the sum over its blocks (1e-12; the energy's bits never change, nodal sums
    add in any order within a block), at every call and at every replay of a
    graph with other calls between."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(elem, n)
    g = np.random.default_rng(n)
    dim = m.X.shape[1]
    u, v = (dev(s * g.standard_normal((m.n_nodes, dim))) for s in (0.01 / n, 1.0))
    mu = dev(np.exp(0.3 * g.standard_normal(m.n_elems)))
    mask = dev((g.random(dim * m.n_nodes) < 0.2).astype(np.uint8))
    a = Operator(elem, m.X, m.conn, block_elems=block, threads=threads)
    b = Operator(elem, m.X, m.conn, block_elems=block, scatter="color")
    for op in (a, b):
        op.set_material(mu, 1.5 * mu)
    calls = (lambda op: op.residual(u), lambda op: op.jacobi_diag(u), lambda op: op.energy(u),
             lambda op: op.hvp(v), lambda op: op.grad_coords(u))
    for mk in (None, mask):
        for op in (a, b):
            op.set_dirichlet(mk)
            op.linearize(u, "f64")
        want = [f(b).cpu() for f in calls]
        psi = calls[2](a).clone()

        def check(outs):
            assert torch.equal(outs[2], psi)
            for got, ref in zip(outs, want):
                assert rel(got.cpu(), ref) <= (1e-12 if ref.dim() == 0 else 1e-11)

        for _ in range(4):
            check([f(a) for f in calls])
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            outs = [f(a) for f in calls]
        for _ in range(4):
            for o in outs:
                o.fill_(7.0)
            graph.replay()
            torch.cuda.synchronize()
            check(outs)
            assert rel(calls[3](a).cpu(), want[3]) <= 1e-11
        for op in (a, b):
            op.linearize(u, "f32")
        assert rel(a.hvp(v.float()).cpu(), b.hvp(v.float()).cpu()) <= 2e-5
    a.close()
    b.close()


@pytest.mark.parametrize("at", [0, 1023, 1024, 1028])
def test_inputs_check_finds_a_moved_coordinate(at):
    """A training step's coordinates, equal to the operator's or off in one
    entry anywhere in the check's slices of 1024 (343 nodes, 1029 entries), with
    a uniform and a varying material in the same wait: energies within 1e-12 of
    the oracle's on those coordinates."""
    from paper_2602_12365_amd import Operator, operator as ops
    m = I.tet_mesh(6)
    g = np.random.default_rng(at)
    u = I.gaussian_field(m.n_nodes, 0.01, 3)
    op = Operator(I.TET4, m.X, m.conn)
    for bump in (0.0, 0.01, 0.0):
        X = m.X.copy()
        X.reshape(-1)[at] += bump
        for mu in (np.full(m.n_elems, 1.25), np.exp(0.3 * g.standard_normal(m.n_elems))):
            before = op.X
            psi = ops.energy(op, dev(u), dev(mu), dev(2.0 * mu), dev(X))
            ref = F.FEM(I.TET4, X, m.conn, mu, 2.0 * mu).energy(u)
            assert abs(float(psi) - ref) <= 1e-12 * abs(ref)
            assert (op.X is before) == bool(torch.equal(before, dev(X)))
    with pytest.raises(TypeError):
        ops.energy(op, dev(u), dev(mu), dev(mu), dev(m.X).float())


@pytest.mark.parametrize("scatter", ["halo", "color", "atomic"])
@pytest.mark.parametrize("elem,n", [(I.HEX8, 9), (I.HEX8, 10), (I.TET4, 9), (I.TET4, 10)])
def test_krylov_on_both_sides_of_one_workgroup(elem, n, scatter):
    """PCG on 1000 nodes (step and direction in one workgroup) and on 1331 (in
    two kernels): FP64 true residuals meet the tolerance (1e-9, and 1e-10 for
    the recursion's drift), FP32 ones 1e-3 (a condition number below 1e4 times
    2^-24), with both preconditioners."""
    from paper_2602_12365_amd import Operator
    m = I.make_mesh(elem, n)
    g = np.random.default_rng(n)
    mu = np.exp(0.3 * g.standard_normal(m.n_elems))
    mask = (m.X[:, 2:] < 1e-9).repeat(3, 1).astype(np.uint8).ravel()
    free = 1.0 - mask.reshape(-1, 3)
    u = 0.005 / n * g.standard_normal((m.n_nodes, 3)) * free
    b = g.standard_normal((m.n_nodes, 3))
    op = Operator(elem, m.X, m.conn, scatter=scatter)
    op.set_material(dev(mu), dev(1.5 * mu))
    op.set_dirichlet(dev(mask))
    orc = F.FEM(elem, m.X, m.conn, mu, 1.5 * mu)
    for precond in (0, 2):
        for prec, rtol, tol in (("f64", 1e-9, 1.1e-9), ("f32", 1e-4, 1e-3)):
            x, it, _ = op.linear_solve(dev(u), dev(b), rtol=rtol, hvp_prec=prec, precond=precond)
            x = x.cpu().numpy()
            assert it > 8 and np.all(x[mask.reshape(-1, 3) == 1] == 0.0)
            assert np.linalg.norm((b - orc.hvp(u, x)) * free) <= tol * np.linalg.norm(b * free)
    op.close()
