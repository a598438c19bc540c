"""GMRES and CG where their vector kernels change: the number of basis columns a kernel takes (1 to 8, then up
to 16, 32 and 64), one and four elements a thread (65,536 unknowns), and the sums of the partials added by the
next kernel or by a launch of their own (524,288 unknowns).

A wrong coefficient spoils the orthogonality of the basis, and the estimate of the residual then parts from the
residual: the solves must stop at the oracle's iteration (+-1: the order of the sums differs), and the
residual, computed here in FP64, must meet the tolerance with 1 % for its own rounding."""
import numpy as np
import pytest

import oracle
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


def residual(s, b, x):
    rows = np.repeat(np.arange(s.n_b), np.diff(s.rp))
    y = np.zeros((s.n_b, 4))
    np.add.at(y, rows, np.einsum("eij,ej->ei", s.val.reshape(-1, 4, 4), x.reshape(-1, 4)[s.ci]))
    return np.linalg.norm(b - y.reshape(-1)) / np.linalg.norm(b)


@pytest.mark.parametrize("nodes,precond,restart", [(700, 1, 63), (700, 1, 20), (700, 0, 9),
                                                   (18e3, 0, 30), (140e3, 0, 30)])
def test_gmres_at_every_kernel_width(scr, nodes, precond, restart):
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    print(f"[gpu] gmres n_b={s.n_b} precond={precond} restart={restart}", flush=True)
    ctx = scr.Context(0)
    h = scr.amg_setup(ctx, scr.SCR_SYSTEM, dev(s.rp), dev(s.ci), dev(s.val.reshape(-1)), dev(s.xyz.reshape(-1)))
    b = synth.rhs(3, 4 * s.n_b, s.mask)
    kw = dict(tol=1e-9, precond=precond, restart=restart, restart_inner=63, tol_A=1e-12, tol_S=1e-12, max_it_A=80, max_it_S=80)
    x = torch.full((4 * s.n_b,), float("nan"), dtype=torch.float64, device="cuda")   # written, not added to
    rc, st = scr.scr_solve(h, dev(b), x, scr.solve_opts(**kw))
    xs = x.cpu().numpy()
    print(f"[gpu] outer {st['outer_it']} its_A {st['its_A']}/{st['calls_A']} its_S {st['its_S']}/{st['calls_S']}", flush=True)
    assert rc == 0 and np.isfinite(xs).all()
    assert residual(s, b, xs) <= 1.01e-9
    if nodes < 1e3:
        o = oracle.Scr(s.rp, s.ci, s.val, s.xyz)
        _, rco, sto = o.solve(b, oracle.solve_opts(**kw))
        assert rco == 0 and abs(st["outer_it"] - sto["outer_it"]) <= 1
    # a tolerance that zero meets, and a right-hand side of zero: x is zero
    x.fill_(float("nan"))
    scr.scr_solve(h, dev(b), x, scr.solve_opts(tol=2.0))
    assert not x.any()
    x.fill_(float("nan"))
    rc, st = scr.scr_solve(h, torch.zeros_like(x), x)
    assert rc == 0 and not x.any()
    h.destroy()
    ctx.destroy()


def test_an_error_inside_a_solve_from_zero_leaves_zero(scr):
    """G scaled by 2^700 and D by 2^-700: S^ is as before, and the right-hand side of the inner velocity solve of
    Algorithm 2 overflows.  The pressure solve around it has not written its result yet and leaves zero."""
    s = synth.generate(synth.default_params(mode=0, m_core=2, n_bl=1, n_wall=1, nz=8, R=1.0, L=2.0))
    ctx = scr.Context(0)
    K = s.val.reshape(-1, 4, 4).copy()
    K[:, :3, 3] *= 2.0 ** 700
    K[:, 3, :3] *= 2.0 ** -700
    print(f"[gpu] error inside a solve n_b={s.n_b}", flush=True)
    h = scr.amg_setup(ctx, scr.SCR_SYSTEM, dev(s.rp), dev(s.ci), dev(K.reshape(-1)), dev(s.xyz.reshape(-1)))
    x = np.zeros(4 * s.n_b)
    x[3 * s.n_b:] = np.random.default_rng(2).uniform(-1, 1, s.n_b)
    y = torch.full((4 * s.n_b,), 7.0, dtype=torch.float64, device="cuda")
    with pytest.raises(scr.ScrError) as e:
        scr.scr_apply(h, "SCR", dev(x), y)
    assert e.value.status == -4
    assert not y[3 * s.n_b:].any()
    h.destroy()
    ctx.destroy()


# Iterations of the same solves with every sum in a launch of its own and every column loaded by itself, the form
# that these kernels were written from; (its_A, its_S, its_I, calls of each)
EXACT = [
    # 3 x 13,344 and 13,344 unknowns: one element a thread; inner bases of 17, 36 and 43 columns
    (700, {}, (64, 72, 1222), (4, 2, 72)),
    (700, dict(cheb_degree=1), (168, 72, 3111), (4, 2, 72)),
    # 3 x 25,242: four elements a thread for the velocity
    (25e3, {}, (62, 79, 1263), (4, 2, 79)),
    (25e3, dict(cheb_degree=1), (160, 79, 3314), (4, 2, 79)),
    # 3 x 204,711: beyond the sums by the next kernel for the velocity; up to 62 columns for the pressure
    (200e3, {}, (95, 125, 3150), (4, 2, 125)),
]


@pytest.mark.parametrize("nodes,amg,its,calls", EXACT)
def test_inner_solves_to_rounding(scr, nodes, amg, its, calls):
    """Inner solves to 1e-11 and 1e-12 make Algorithm 1 an exact preconditioner: two outer iterations, and the
    iterations of each inner solve as above (+-1 a solve: the order of the sums differs).  A wrong coefficient for
    one width of the basis shows in the first or in the second."""
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    print(f"[gpu] inner solves n_b={s.n_b} {amg}", flush=True)
    ctx = scr.Context(0)
    h = scr.amg_setup(ctx, scr.SCR_SYSTEM, dev(s.rp), dev(s.ci), dev(s.val.reshape(-1)), dev(s.xyz.reshape(-1)),
                      scr.amg_opts(**amg))
    b = synth.rhs(3, 4 * s.n_b, s.mask)
    x = torch.empty(4 * s.n_b, dtype=torch.float64, device="cuda")
    rc, st = scr.scr_solve(h, dev(b), x, scr.solve_opts(tol=1e-9, tol_A=1e-12, tol_S=1e-11, tol_I=1e-12, restart_inner=63,
                                                        max_it_A=300, max_it_S=300, max_it_I=300))
    got = [(st["its_" + k], st["calls_" + k]) for k in "ASI"]
    print(f"[gpu] outer {st['outer_it']} (iterations, solves) {got}", flush=True)
    assert rc == 0 and st["outer_it"] == 2
    assert residual(s, b, x.cpu().numpy()) <= 1e-11
    for (i, n), ref, nref in zip(got, its, calls):
        assert i / n > 8 and abs(i / n - ref / nref) <= 1
    h.destroy()
    ctx.destroy()


# one element a thread, four, the longest vectors whose partials the next kernel adds, and beyond
@pytest.mark.parametrize("nodes,n,its", [(60e3, 54777, 12), (100e3, 109512, 13), (300e3, 308550, 14), (600e3, 570103, 15)])
@pytest.mark.parametrize("precision", [0, 1])
def test_cg_at_every_grid(scr, nodes, n, its, precision):
    """CG (precision 0) and flexible CG (1) on the three columns: the iterations of the form with a launch for each
    sum (+-1), the residual of the recurrence and the true one at the tolerance; a column that is done (zero) stays."""
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    assert s.n_phys == n
    print(f"[gpu] cg n={n} precision={precision}", flush=True)
    ctx = scr.Context(0)
    h = scr.amg_setup(ctx, scr.MESH_SYSTEM, dev(s.Lrp), dev(s.Lci), dev(s.Lval), None, scr.amg_opts(precision=precision))
    b = synth.rhs(31, 3 * n, np.repeat(s.Lmask, 3)).reshape(-1, 3)
    b[:, 1] *= 1e-3
    rows = np.repeat(np.arange(n), np.diff(s.Lrp))
    for cols in ((0, 1, 2), (0, 2)):
        bb = np.zeros_like(b)
        bb[:, cols] = b[:, cols]
        x = torch.full((3 * n,), float("nan"), dtype=torch.float64, device="cuda")
        rc, st = scr.mesh_motion_solve(h, dev(bb.reshape(-1)), x, scr.solve_opts(tol=1e-10))
        xs = x.cpu().numpy().reshape(-1, 3)
        assert rc == 0
        for c in range(3):
            if c not in cols:
                assert st["mesh_its"][c] == 0 and not xs[:, c].any()
                continue
            r = bb[:, c] - np.bincount(rows, weights=s.Lval * xs[s.Lci, c], minlength=n)
            assert abs(st["mesh_its"][c] - its) <= 1
            assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(bb[:, c])
    h.destroy()
    ctx.destroy()
