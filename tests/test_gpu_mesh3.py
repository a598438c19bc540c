"""The V-cycle of AMG(L) on the three columns of a mesh solve against the one-column V-cycle, bit for bit.  One
iteration of CG from zero leaves x = alpha (V-cycle of b) in every column, each entry rounded once, so the bits of
the three-column cycle show through one alpha per column."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def scr():
    import paper_2206_06996_amd.scr as m
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# coarsest levels of every remainder of the 512 columns that the dense product takes at a time, and restrictions
# with one and with four wavefronts per row
@pytest.mark.parametrize("nodes,coarse_max", [(700, 0), (700, 100), (25e3, 0), (25e3, 40), (140e3, 0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_columns_bitwise_the_one_column_cycle(scr, nodes, coarse_max, precision):
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    print(f"[gpu] mesh columns n={s.n_phys} precision={precision} coarse_max={coarse_max}", flush=True)
    ctx = scr.Context(0)
    kw = dict(coarse_max=coarse_max) if coarse_max else {}
    h = scr.amg_setup(ctx, scr.MESH_SYSTEM, dev(s.Lrp), dev(s.Lci), dev(s.Lval), None, scr.amg_opts(precision=precision, **kw))
    info = [h.hier_level_info(2, l) for l in range(h.hier_levels(2))]
    if nodes == 25e3:
        assert any(0 < i["nagg"] < 2048 and i["nnzR"] >= 64 * i["nagg"] for i in info)
    b = synth.rhs(31, 3 * s.n_phys, np.repeat(s.Lmask, 3))
    x = torch.zeros(3 * s.n_phys, dtype=torch.float64, device="cuda")
    scr.mesh_motion_solve(h, dev(b), x, scr.solve_opts(tol=1e-30, max_it=1))
    xs = x.cpu().numpy()
    for c in range(3):
        z = torch.empty(s.n_phys, dtype=torch.float64, device="cuda")
        scr.scr_apply(h, "VL", dev(b[c::3]), z)
        z, xc = z.cpu().numpy(), xs[c::3]
        k = np.argmax(np.abs(z))
        a = xc[k] / z[k]
        alphas = [a + u * np.spacing(a) for u in range(-3, 4)]
        wrong = min(np.count_nonzero(xc != al * z) for al in alphas)
        assert wrong == 0, (c, wrong, s.n_phys)
    h.destroy()
    ctx.destroy()


# the classical kind: hybrid Gauss-Seidel sweeps of up to 1,024 domains of 64 rows, and of more
@pytest.mark.parametrize("nodes", [700, 25e3, 140e3])
@pytest.mark.parametrize("precision", [0, 1])
def test_classical_columns_bitwise_the_one_column_cycle(scr, nodes, precision):
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    print(f"[gpu] classical mesh columns n={s.n_phys} precision={precision}", flush=True)
    ctx = scr.Context(0)
    h = scr.amg_setup(ctx, scr.MESH_SYSTEM, dev(s.Lrp), dev(s.Lci), dev(s.Lval), None,
                      scr.amg_opts(amg_type=1, precision=precision))
    b = synth.rhs(31, 3 * s.n_phys, np.repeat(s.Lmask, 3))
    x = torch.zeros(3 * s.n_phys, dtype=torch.float64, device="cuda")
    scr.mesh_motion_solve(h, dev(b), x, scr.solve_opts(tol=1e-30, max_it=1))
    xs = x.cpu().numpy()
    for c in range(3):
        z = torch.empty(s.n_phys, dtype=torch.float64, device="cuda")
        scr.scr_apply(h, "VL", dev(b[c::3]), z)
        z, xc = z.cpu().numpy(), xs[c::3]
        k = np.argmax(np.abs(z))
        a = xc[k] / z[k]
        wrong = min(np.count_nonzero(xc != (a + u * np.spacing(a)) * z) for u in range(-3, 4))
        assert wrong == 0, (c, wrong, s.n_phys)
    h.destroy()
    ctx.destroy()


# a grid whose last row couples to `longest` - 1 nodes: both sides of the length that changes the sweeps
@pytest.mark.parametrize("longest", [511, 512, 4097])
@pytest.mark.parametrize("amg_type", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_columns_bitwise_with_a_long_row(scr, longest, amg_type, precision):
    sps = pytest.importorskip("scipy.sparse")
    n, eps = 64, 1e-3
    T = sps.diags([-np.ones(n - 1), 2 * np.ones(n), -np.ones(n - 1)], [-1, 0, 1])
    L = sps.kron(sps.identity(n), T) + sps.kron(T, sps.identity(n))
    w = np.where(np.arange(n * n) < longest - 1, eps, 0.0)
    B = sps.csr_matrix(-w[:, None])
    B.eliminate_zeros()
    A = sps.bmat([[L + sps.diags(w), B], [B.T, sps.csr_matrix([[w.sum() + 1.0]])]], format="csr")
    A.sort_indices()
    N = A.shape[0]
    assert np.diff(A.indptr).max() == longest
    print(f"[gpu] mesh columns, longest row {longest} kind={amg_type} precision={precision}", flush=True)
    ctx = scr.Context(0)
    h = scr.amg_setup(ctx, scr.MESH_SYSTEM, dev(A.indptr.astype(np.int32)), dev(A.indices.astype(np.int32)), dev(A.data),
                      None, scr.amg_opts(amg_type=amg_type, precision=precision))
    b = synth.rhs(31, 3 * N)
    x = torch.zeros(3 * N, dtype=torch.float64, device="cuda")
    scr.mesh_motion_solve(h, dev(b), x, scr.solve_opts(tol=1e-30, max_it=1))
    xs = x.cpu().numpy()
    for c in range(3):
        z = torch.empty(N, dtype=torch.float64, device="cuda")
        scr.scr_apply(h, "VL", dev(b[c::3]), z)
        z, xc = z.cpu().numpy(), xs[c::3]
        k = np.argmax(np.abs(z))
        a = xc[k] / z[k]
        wrong = min(np.count_nonzero(xc != (a + u * np.spacing(a)) * z) for u in range(-3, 4))
        assert wrong == 0, (c, wrong, N)
    h.destroy()
    ctx.destroy()
