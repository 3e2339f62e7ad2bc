"""Dyadic level sums against the oracle where their plans take another path:
fewer bisections of the panels than the level's number, and candidate lists
cut into pieces (one batch, several, a ragged last one).

Densities are random at every node, the worst that a panel's interpolant can
hold.  The sums must agree with the oracle's j bisections to tol of the
largest level sum: the rule admits tol/100 of the kernel per source.
"""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("panels,dx,tol,n", [(32, 0.1, 1e-10, 1), (64, 0.1, 1e-10, 63), (96, 0.1, 1e-6, 64),
                                             (160, 0.08, 1e-12, 65), (32, 0.03, 1e-10, 700)])
def test_random_densities(panels, dx, tol, n):
    import paper_2606_28865_amd as M
    print(f"case panels={panels} dx={dx} tol={tol} n={n}", flush=True)
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], panels)
    g = np.random.default_rng(panels + n)
    # targets within a few level radii of the boundary, on both sides
    i = g.integers(0, 16 * panels, n)
    d = g.normal(0.0, dx, n)
    tx, ty = bnd["x"][i] + d * bnd["nx"][i], bnd["y"][i] + d * bnd["ny"][i]
    inside = (d < 0).astype(np.int8)
    sigma, mu = g.standard_normal((2, 16 * panels))
    plan = M.Plan(M.make_params(alpha=5.0, tol=tol, dx=dx), bnd, None, (tx, ty, inside), on_surface=True)
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    S, D, _ = plan.eval(dev(sigma), dev(mu), parts=M.PART_LEVELS)
    torch.cuda.synchronize()
    ref = O.Problem(5.0, plan.info()["delta"], 3, bnd, targets=(tx, ty), inside=inside, on_surface=True, sigma=sigma,
                    mu=mu, parts=O.PART_LEVELS).eval()
    for name, a, b in (("S", S, ref[0]), ("D", D, ref[1])):
        err = np.abs(a.cpu().numpy().ravel() - b).max() / np.abs(b).max()
        print(f"{name}: {err:.2e}", flush=True)
        assert err < tol, (name, err)
