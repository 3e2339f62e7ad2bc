"""Dyadic level sums on few, strongly curved panels, where the panels are short
enough for fewer bisections of a straight panel but the curve and its uneven
speed are not: the sums must still agree with the oracle's j bisections to tol
of the largest level sum, for densities that are random at every node (the
plan's rule bounds the error by tol/10 of the kernel per source).  The last
four take fewer bisections with the rule's bound near its limit.
"""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("panels,dx,tol", [(32, 0.125, 1e-10), (24, 0.17, 1e-10), (32, 0.149, 1e-12),
                                           (96, 0.122, 1e-10), (64, 0.09, 1e-6),
                                           (96, 0.054, 1e-10), (64, 0.0563, 1e-6)])
def test_random_densities(panels, dx, tol):
    import paper_2606_28865_amd as M
    print(f"case panels={panels} dx={dx} tol={tol}", flush=True)
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], panels)
    g = np.random.default_rng(panels)
    i = g.integers(0, 16 * panels, 200)
    d = g.normal(0.0, dx, 200)
    tx, ty = bnd["x"][i] + d * bnd["nx"][i], bnd["y"][i] + d * bnd["ny"][i]
    inside = (d < 0).astype(np.int8)
    sigma, mu = g.standard_normal((2, 16 * panels))
    plan = M.Plan(M.make_params(alpha=5.0, tol=tol, dx=dx), bnd, None, (tx, ty, inside), on_surface=True)
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    S, D, _ = plan.eval(dev(sigma), dev(mu), parts=M.PART_LEVELS)
    torch.cuda.synchronize()
    ref = O.Problem(5.0, plan.info()["delta"], 3, bnd, targets=(tx, ty), inside=inside, on_surface=True, sigma=sigma,
                    mu=mu, parts=O.PART_LEVELS).eval()
    plan.close()
    for name, a, b in (("S", S, ref[0]), ("D", D, ref[1])):
        err = np.abs(a.cpu().numpy().ravel() - b).max() / np.abs(b).max()
        print(f"{name}: {err:.2e}", flush=True)
        assert err < tol, (name, err)
