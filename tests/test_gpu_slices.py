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
