"""Evaluations of some of the potentials only: each equals the same potential
of the joint evaluation (the same sums in the same order: the history fields
are transformed independently), also after an evaluation that left other
values in the plan's grids."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,batch,delta", [("f64", 1, 0.0), ("f32", 3, 0.0), ("f64", 1, 2e-6)])
def test_subsets_equal_joint(prec, batch, delta):
    import paper_2606_28865_amd as M
    w = synth.config0(grid=24)
    f32 = prec == "f32"
    # delta 2e-6: a grid beyond 8192 points, through the 2D transforms
    plan = M.Plan(M.make_params(alpha=10.0, tol=1e-6 if f32 else 1e-10, dx=w.dx, delta=delta, batch=batch,
                                prec=M.MHK_FP32 if f32 else M.MHK_FP64), w.boundary, w.volume,
                  (w.tx, w.ty, w.inside), on_surface=True)
    g = np.random.default_rng(3)
    dev = lambda a: torch.as_tensor(np.stack([a * g.uniform(0.5, 2.0) for _ in range(batch)]),
                                    dtype=torch.float32 if f32 else torch.float64, device="cuda")
    sig, mu, fv, ft = dev(w.sigma), dev(w.mu), dev(w.f_vol), dev(w.f_trg)
    joint = [o.clone() for o in plan.eval(sig, mu, fv, ft)]
    for keep in ("S", "D", "V", "SD", "SV", "DV"):
        print(f"case {prec} batch {batch} delta {delta}: {keep}", flush=True)
        plan.eval(3.0 * sig, -2.0 * mu, 5.0 * fv, ft)
        out = plan.eval(sig if "S" in keep else None, mu if "D" in keep else None, fv if "V" in keep else None,
                        ft if "V" in keep else None)
        torch.cuda.synchronize()
        for c, o, j in zip("SDV", out, joint):
            if c not in keep:
                assert o is None
                continue
            m = torch.isfinite(j)
            assert torch.equal(m, torch.isfinite(o))
            err = (o[m] - j[m]).abs().max() / j[m].abs().max()
            assert err < (1e-6 if f32 else 1e-13), (keep, c, float(err))
