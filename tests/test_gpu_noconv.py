"""Plans whose targets lie in a local band next to a centre of curvature, where
the distance is flat and the closest point's parameter is found to no better
than 1e-12, are refused with MHK_ENOCONV; the same circle with targets off its
centre is accepted, and its S and D agree with the oracle to ten times tol."""
import numpy as np
import pytest

import oracle as O
import synth
from helpers import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _circle(r, n):
    """A circle off the origin (so that the nodes are rounded), and n targets at distance r from its centre."""
    cv = synth.Curve(r0=0.3, cx=0.37, cy=-0.21)
    t = 2 * np.pi * np.random.default_rng(1).random(n)
    return synth.discretize([cv], 12), (cv.cx + r * np.cos(t), cv.cy + r * np.sin(t), np.ones(n, np.int8))


PRM = dict(alpha=2.0, tol=1e-10, delta=0.05, J=2)


@pytest.mark.parametrize("r", [1e-6, 1e-5, 10 ** -4.5])
def test_centre_of_curvature_refused(r):
    import paper_2606_28865_amd as M
    assert M.resolve_params(**PRM)["band_layer"] > 0.3
    print(f"case targets at a centre of curvature, r={r}", flush=True)
    bnd, tg = _circle(r, 20000)
    with pytest.raises(M.MhkError) as e:
        M.Plan(M.make_params(**PRM), bnd, None, tg, on_surface=False)
    assert e.value.code == -5


@pytest.mark.parametrize("r", [0.05, 0.2])
def test_off_centre_accepted(r):
    import paper_2606_28865_amd as M
    print(f"case targets at radius {r}", flush=True)
    bnd, (tx, ty, ins) = _circle(r, 200)
    plan = M.Plan(M.make_params(**PRM), bnd, None, (tx, ty, ins), on_surface=False)
    t = bnd["t"]
    sigma, mu = 1 + 0.3 * np.cos(3 * t), np.sin(2 * t)
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    S, D, _ = plan.eval(dev(sigma), dev(mu))
    torch.cuda.synchronize()
    ref = O.Problem(2.0, plan.info()["delta"], 2, bnd, targets=(tx, ty), inside=ins, on_surface=False, sigma=sigma,
                    mu=mu).eval()
    plan.close()
    assert rel_err(S.cpu().numpy(), ref[0]) < 1e-9
    assert rel_err(D.cpu().numpy(), ref[1]) < 1e-9
