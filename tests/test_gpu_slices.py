"""Sliced-ELL kernels over the sizes at which their split of a slice's work changes: wavefronts per slice
(block-row lanes: 8 from 209 slices, 4 at 395, 2 at about 1,550, 1 above 2,048) and, on the coarse levels,
the row positions that share a row (1 to 16 of a 1x1 slice, 1, 2 and 5 of a 6x6 one).

Against the FP64 oracle with the bars of the other parity tests: products within 1e-13 of the largest entry
(rows of at most 30 blocks, FMA against unfused rounding), FP64 V-cycles within 1e-10, FP32 ones within 1e-4."""
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


@pytest.mark.parametrize("nodes", [700, 13e3, 25e3, 95e3, 140e3])
def test_products_and_vcycles_at_every_split(scr, nodes):
    s = synth.generate(synth.tube_params(nodes, 1.0, 5.0))
    print(f"[gpu] slices n_b={s.n_b}", flush=True)
    ctx = scr.Context(0)
    o = oracle.Scr(s.rp, s.ci, s.val, s.xyz)
    rng = np.random.default_rng(int(nodes))
    xs = {op: rng.uniform(-1, 1, k * s.n_b) for op, k in (("A", 3), ("G", 1), ("D", 3), ("C", 1), ("Shat", 1), ("VA", 3), ("VS", 1))}
    for precision in (scr.SCR_FP64, scr.SCR_MIXED):
        h = scr.amg_setup(ctx, scr.SCR_SYSTEM, dev(s.rp), dev(s.ci), dev(s.val.reshape(-1)), dev(s.xyz.reshape(-1)),
                          scr.amg_opts(precision=precision))
        for op, x in xs.items():
            yo = o.apply(op, x)
            y = torch.empty(yo.size, dtype=torch.float64, device="cuda")
            scr.scr_apply(h, op, dev(x), y)
            d = y.cpu().numpy() - yo
            if op in ("VA", "VS"):
                bar = 1e-10 if precision == scr.SCR_FP64 else 1e-4
                assert np.linalg.norm(d) <= bar * np.linalg.norm(yo), (op, precision)
            else:
                assert np.abs(d).max() <= 1e-13 * np.abs(yo).max(), (op, precision)
        h.destroy()
    ctx.destroy()


def test_setup_products_on_a_shuffled_numbering(scr):
    """Rows renumbered at random: the columns of a product's row then span the whole matrix (about 42,000
    columns), beyond the 8,192 and 32,768 that its maps hold at a time.  Patterns, aggregates and strength
    flags bit-exact against the oracle, values within the bars of the hierarchy tests."""
    from tests.test_gpu_parity import _compare_hierarchy
    s = synth.generate(synth.tube_params(40e3, 1.0, 5.0))
    n = s.n_b
    assert n > 32768
    new = np.random.default_rng(1).permutation(n)                # new index of each row
    rows = np.repeat(np.arange(n), np.diff(s.rp))
    r, c = new[rows], new[s.ci]
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(np.bincount(r, minlength=n))
    ci, val = c[order].astype(np.int32), s.val[order]
    xyz = np.empty_like(s.xyz)
    xyz[new] = s.xyz
    ctx = scr.Context(0)
    print(f"[gpu] shuffled setup n_b={n}", flush=True)
    h = scr.amg_setup(ctx, scr.SCR_SYSTEM, dev(rp), dev(ci), dev(val.reshape(-1)), dev(xyz.reshape(-1)))
    o = oracle.Scr(rp, ci, val, xyz)
    grp, gci, gv = h.matrix_copy("Shat")
    orp, oci, ov = o.matrix("Shat")
    assert np.array_equal(grp, orp) and np.array_equal(gci, oci)
    assert np.abs(gv - ov).max() <= 1e-13 * np.abs(ov).max()
    _compare_hierarchy(h, 0, o.amgA)
    _compare_hierarchy(h, 1, o.amgS)
    h.destroy()
    ctx.destroy()
