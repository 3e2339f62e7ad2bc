"""The history part's interpolation on each of its paths, against the oracle's
history sums: blocks of dense targets on the matrix cores (block edges 8 and 4,
ragged counts about 16 and 32 per block), tiles, and few targets far apart; the
window widths at which the path changes.  The bar is the plan's tolerance of
the largest history value."""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,box,tol,dx", [(1, 1.4, 1e-10, 0.1), (15, 0.02, 1e-10, 0.1), (33, 0.02, 1e-10, 0.1),
                                          (200, 0.1, 1e-5, 0.1), (900, 0.3, 1e-7, 0.1), (500, 0.2, 1e-8, 0.1),
                                          (700, 0.3, 1e-10, 0.1), (400, 0.1, 1e-11, 0.1), (400, 0.1, 1e-12, 0.1),
                                          (40, 1.4, 1e-10, 0.02), (3000, 1.4, 1e-10, 0.02)])
def test_history_at_targets(n, box, tol, dx):
    import paper_2606_28865_amd as M
    print(f"case n={n} box={box} tol={tol} dx={dx}", flush=True)
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], 48)
    g = np.random.default_rng(n)
    tx, ty = g.uniform(-box, box, n), g.uniform(-box, box, n)
    inside = (np.hypot(tx, ty) < 1 + 0.3 * np.cos(5 * np.arctan2(ty, tx))).astype(np.int8)
    k = np.arange(5)[:, None] * bnd["t"]
    sigma, mu = g.standard_normal(5) @ np.cos(k), g.standard_normal(5) @ np.sin(k + 0.3)
    plan = M.Plan(M.make_params(alpha=3.0, tol=tol, dx=dx), bnd, None, (tx, ty, inside))
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    S, D, _ = plan.eval(dev(sigma), dev(mu), parts=M.PART_HISTORY)
    torch.cuda.synchronize()
    ref = O.Problem(3.0, plan.info()["delta"], 3, bnd, targets=(tx, ty), inside=inside, sigma=sigma, mu=mu,
                    parts=O.PART_HISTORY).eval()
    big = [np.abs(O.GH(0.0, 3.0, plan.info()["delta"])) * np.abs(bnd["w"] * s).sum() for s in (sigma, mu)]
    for name, a, b, sc in (("S", S, ref[0], big[0]), ("D", D, ref[1], big[1])):
        err = np.abs(a.cpu().numpy().ravel() - b).max() / max(np.abs(b).max(), 1e-3 * sc)
        print(f"{name}: {err:.2e} (W = {plan.info()['wspread']}, n = {plan.info()['n_fine']})", flush=True)
        assert err < 2 * tol, (name, err)
