"""Level sums of several densities (from five on in groups of 16 on the matrix
cores) against the same plan's sums of one density: the same kernel values summed
in another order, so the difference is rounding of FP64 sums of up to some
thousand terms."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n,what", [(4, 300, "SD"), (5, 1, "SD"), (8, 63, "S"), (15, 65, "D"), (16, 700, "SD"),
                                          (17, 130, "SD"), (33, 64, "SD")])
def test_batch_equals_single(batch, n, what):
    import paper_2606_28865_amd as M
    print(f"case batch={batch} n={n} {what}", flush=True)
    bnd = synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], 64)
    g = np.random.default_rng(batch + n)
    i = g.integers(0, 1024, n)
    d = g.normal(0.0, 0.05, n)
    tx, ty = bnd["x"][i] + d * bnd["nx"][i], bnd["y"][i] + d * bnd["ny"][i]
    inside = (d < 0).astype(np.int8)
    q = torch.as_tensor(g.standard_normal((2, batch, 1024)), device="cuda")
    mk = lambda b: M.Plan(M.make_params(alpha=5.0, tol=1e-10, dx=0.1, batch=b), bnd, None, (tx, ty, inside),
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
            assert err < 1e-13, (w, b, err)
    plan.close()
    one.close()
