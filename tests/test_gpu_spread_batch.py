"""Spreading of batches: one density per workgroup where the blocks are few
(16, 8 or 4 wavefronts by their number) and several beyond, at both precisions
and up to the widest window (16 wavefronts of it use all of a CU's LDS).  The
history part of a batch equals that of each density alone, whose sums are the
same but for their order; and the widest window agrees with the narrower one."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _history(w, batch, dens, prec, **kw):
    import paper_2606_28865_amd as M
    plan = M.Plan(M.make_params(alpha=10.0, tol=1e-6 if prec else 1e-10, batch=batch, prec=prec, **kw), w.boundary,
                  w.volume, (w.tx, w.ty, w.inside), on_surface=True)
    out = [o.cpu().numpy().astype(np.float64) for o in plan.eval(*dens, parts=M.PART_HISTORY)]
    torch.cuda.synchronize()
    plan.close()
    return out


# delta and with it the grid: from some ten blocks with sources to a few
# thousand (one each, 16, 8 and 4 wavefronts, then by eights)
@pytest.mark.parametrize("delta", [1e-2, 1e-3, 2e-4, 2e-5])
@pytest.mark.parametrize("batch,prec,wspread", [(2, 0, 0), (3, 1, 0), (5, 0, 0), (9, 1, 0), (2, 0, 16), (8, 0, 16)])
def test_batch_equals_single(delta, batch, prec, wspread):
    print(f"case batch {batch} prec {prec} wspread {wspread} delta {delta}", flush=True)
    w = synth.multibody(cfg=11, n_bodies=3, n_boundary=2048, n_volume=20000, n_targets=500, box=0.6)
    g = np.random.default_rng(batch)
    dt = torch.float32 if prec else torch.float64
    dev = lambda a: torch.as_tensor(np.stack([a * g.uniform(0.5, 2.0) for _ in range(batch)]), dtype=dt, device="cuda")
    dens = [dev(a) for a in (w.sigma, w.mu, w.f_vol, w.f_trg)]
    got = _history(w, batch, dens, prec, delta=delta, wspread=wspread)
    for b in (0, batch - 1):
        one = _history(w, 1, [d[b:b + 1].contiguous() for d in dens], prec, delta=delta, wspread=wspread)
        for name, a, r in zip("SDV", got, one):
            # 64-bit sums in another order; FP32 transforms round once more per grid value
            assert np.abs(a[b] - r[0]).max() <= (1e-6 if prec else 1e-13) * np.abs(r[0]).max(), name


@pytest.mark.parametrize("n_volume", [20000, 200000])
def test_widest_window(n_volume):
    """wspread = 16, one density: 16 wavefronts on few blocks, 8 or 4 on more."""
    w = synth.multibody(cfg=11, n_bodies=3, n_boundary=2048, n_volume=n_volume, n_targets=500, box=0.6)
    print(f"case widest window, {n_volume} volume nodes", flush=True)
    dens = [torch.as_tensor(a[None], dtype=torch.float64, device="cuda") for a in (w.sigma, w.mu, w.f_vol, w.f_trg)]
    for delta in (1e-2, 1e-3, 2e-4):
        a = _history(w, 1, dens, 0, delta=delta, wspread=16)
        r = _history(w, 1, dens, 0, delta=delta)
        for name, x, y in zip("SDV", a, r):
            assert np.abs(x - y).max() <= 1e-9 * np.abs(y).max(), (delta, name)   # both err by tol = 1e-10
