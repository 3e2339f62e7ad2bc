"""mhk_plan_footprint, which admits plans to the server's memory budget, is no
less than the device bytes that the plan then owns: few targets with long
candidate lists (many level items per target wavefront), batches, volume levels,
FP32, layer potentials alone, and a plan whose small buffers share one chunk."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# bodies, boundary nodes, volume nodes, targets, plan parameters
CASES = [(3, 49152, 0, 2000, dict(batch=16, delta=1e-2)),
         (3, 16384, 0, 100, dict(batch=64, delta=1e-2)),
         (3, 2048, 40000, 6000, dict(batch=1, dx=0.02, v_levels=1)),
         (3, 2048, 40000, 500, dict(batch=3, delta=2e-3, v_levels=1)),
         (3, 8192, 40000, 50000, dict(batch=8, delta=1e-3, prec=1, tol=1e-6)),
         (1, 512, 0, 70, dict(batch=1, delta=1e-2))]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_footprint_covers_plan(case):
    import paper_2606_28865_amd as M
    n_bodies, nb, nv, nt, kw = CASES[case]
    print(f"case {CASES[case]}", flush=True)
    w = synth.multibody(cfg=11, n_bodies=n_bodies, n_boundary=nb, n_volume=max(nv, 5000), n_targets=nt, box=0.6)
    prm = M.make_params(**dict(dict(alpha=10.0, tol=1e-10), **kw))
    geo = (w.boundary, w.volume if nv else None, (w.tx, w.ty, w.inside))
    need = M.footprint(prm, *geo, on_surface=False)
    plan = M.Plan(prm, *geo, on_surface=False)
    got = plan.info()["device_bytes"]
    plan.close()
    print(f"footprint {need / 2**20:.1f} MiB, plan {got / 2**20:.1f} MiB", flush=True)
    assert need >= got
