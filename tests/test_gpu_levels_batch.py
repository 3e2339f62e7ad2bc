"""Level sums of several densities (from five on in groups of 16 on the matrix
cores) against the same plan's sums of one density: the same kernel values summed
in another order, so the difference is rounding of FP64 sums of up to some
thousand terms; in FP32 that of the single density's sums of 64 terms in FP32,
64 times 2^-24 of partial sums up to five times the largest sum."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("batch,n,what", [(4, 300, "SD"), (5, 1, "SD"), (8, 63, "S"), (15, 65, "D"), (16, 700, "SD"),
                                          (17, 130, "SD"), (33, 64, "SD")])
def test_batch_equals_single(batch, n, what, prec):
    import paper_2606_28865_amd as M
    print(f"case batch={batch} n={n} {what} {prec}", flush=True)
    f32 = prec == "f32"
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], 64)
    g = np.random.default_rng(batch + n)
    i = g.integers(0, 1024, n)
    d = g.normal(0.0, 0.05, n)
    tx, ty = bnd["x"][i] + d * bnd["nx"][i], bnd["y"][i] + d * bnd["ny"][i]
    inside = (d < 0).astype(np.int8)
    q = torch.as_tensor(g.standard_normal((2, batch, 1024)), dtype=torch.float32 if f32 else torch.float64,
                        device="cuda")
    mk = lambda b: M.Plan(M.make_params(alpha=5.0, tol=1e-6 if f32 else 1e-10, dx=0.1, batch=b,
                                        prec=M.MHK_FP32 if f32 else M.MHK_FP64), bnd, None, (tx, ty, inside),
                          on_surface=True)
    plan, one = mk(batch), mk(1)
    many = plan.eval(*[q[c] if w in what else None for c, w in enumerate("SD")], parts=M.PART_LEVELS)
    torch.cuda.synchronize()
    for b in range(batch):
        ref = one.eval(*[q[c, b] if w in what else None for c, w in enumerate("SD")], parts=M.PART_LEVELS)
        torch.cuda.synchronize()
        for c, w in enumerate("SD"):
            if w not in what:
                continue
            a, r = many[c][b].ravel(), ref[c].ravel()
            err = float((a - r).abs().max() / r.abs().max())
            assert err < (2e-5 if f32 else 1e-13), (w, b, err)
    plan.close()
    one.close()
