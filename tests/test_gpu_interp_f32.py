"""The FP32 history part's interpolation against the oracle's history sums of the
same (FP32) densities: blocks on the matrix cores, whose FP32 results lie in
other rows than the FP64 ones, tiles, and few targets far apart; batches of more
densities than a wavefront takes.  The bar is twice the plan's tolerance of
the largest history value."""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-6


@pytest.mark.parametrize("n,box,dx,batch", [(15, 0.02, 0.1, 1), (33, 0.02, 0.1, 1), (200, 0.1, 0.1, 5),
                                            (900, 0.3, 0.1, 4), (2500, 0.3, 0.1, 1), (40, 1.4, 0.02, 2),
                                            (3000, 1.4, 0.02, 1), (6000, 1.4, 0.05, 9)])
def test_history_at_targets(n, box, dx, batch):
    import paper_2606_28865_amd as M
    print(f"case n={n} box={box} dx={dx} batch={batch}", flush=True)
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], 48)
    g = np.random.default_rng(n)
    tx, ty = g.uniform(-box, box, n), g.uniform(-box, box, n)
    inside = (np.hypot(tx, ty) < 1 + 0.3 * np.cos(5 * np.arctan2(ty, tx))).astype(np.int8)
    k = np.arange(5)[:, None] * bnd["t"]
    sigma = (g.standard_normal((batch, 5)) @ np.cos(k)).astype(np.float32)
    mu = (g.standard_normal((batch, 5)) @ np.sin(k + 0.3)).astype(np.float32)
    plan = M.Plan(M.make_params(alpha=3.0, tol=TOL, dx=dx, prec=M.MHK_FP32, batch=batch), bnd, None, (tx, ty, inside))
    S, D, _ = plan.eval(torch.as_tensor(sigma, device="cuda"), torch.as_tensor(mu, device="cuda"),
                        parts=M.PART_HISTORY)
    torch.cuda.synchronize()
    delta = plan.info()["delta"]
    for b in {0, batch - 1}:
        s, m = sigma[b].astype(np.float64), mu[b].astype(np.float64)
        ref = O.Problem(3.0, delta, 3, bnd, targets=(tx, ty), inside=inside, sigma=s, mu=m,
                        parts=O.PART_HISTORY).eval()
        gh = np.abs(O.GH(0.0, 3.0, delta))
        for name, a, r, q in (("S", S, ref[0], s), ("D", D, ref[1], m)):
            # (no less than a tenth of the sources' absolute sum: what FP32 sums round to)
            err = np.abs(a[b].cpu().numpy() - r).max() / max(np.abs(r).max(), 0.1 * gh * np.abs(bnd["w"] * q).sum())
            print(f"{name}: {err:.2e} (W = {plan.info()['wspread']}, n = {plan.info()['n_fine']})", flush=True)
            assert err < 2 * TOL, (name, err)
    plan.close()
