"""Nystrom products that keep no partial sums in their object (whole rows from
the triangle, two launches otherwise): recorded into a graph at sizes around the
edges of their launch shapes, with remainders of 16 to 112 nodes in the last tile
column; of few nodes; and of two threads that share the per-thread stream's
handle.  Compared with eager products of the triangle, which other tests
compare with the dense matrix of the oracle, and of few nodes with that."""
import threading

import numpy as np
import pytest

import synth
from helpers import rel_err
from oracle import bie

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# sums of at most 12352 terms in another order, 12352 eps = 1.4e-12 of their
# absolute sums at worst; random signs leave about the root of that
TOL = 1e-12


def _boundary(panels):
    return synth.discretize([synth.Curve(r0=1.0, a=0.3, l1=5)], panels)


@pytest.mark.parametrize("panels", [129, 192, 193, 256, 257, 260, 263, 512, 513, 768, 772])
def test_captured(panels):
    import paper_2606_28865_amd as M
    n = 16 * panels
    print(f"case captured product n={n}", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        nys = M.Nystrom(3.0, _boundary(panels))
        g = torch.Generator(device="cuda").manual_seed(panels)
        x = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
        out = torch.empty_like(x)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            nys.apply(x, shift=0.5, out=out)
        for k in (None, 0, 63, 64, 127, 128, n - 1):
            x.normal_(generator=g)
            if k is not None:
                x[k] = np.inf                    # its column alone is infinite, and nothing a NaN beside row k
            out.fill_(float("nan"))
            graph.replay()
            ref = nys.apply(x, shift=0.5)
            st.synchronize()
            a, b = out.cpu().numpy(), ref.cpu().numpy()
            if k is None:
                assert rel_err(a, b) < TOL
            else:
                np.testing.assert_array_equal(a, b)
                assert np.isinf(np.delete(a, k)).all()
    nys.close()


@pytest.mark.parametrize("panels", [1, 4, 5, 8, 9, 127, 128, 129])
def test_few_nodes(panels):
    import paper_2606_28865_amd as M
    n = 16 * panels
    print(f"case product n={n}", flush=True)
    bnd = _boundary(panels)
    K = bie.nystrom_matrix(bnd, 3.0)
    nys = M.Nystrom(3.0, bnd)
    x = np.random.default_rng(panels).standard_normal(n)
    y = nys.apply(torch.as_tensor(x, device="cuda"), shift=-0.5).cpu().numpy()
    # n sums of at most n terms, elements to a few eps
    assert np.abs(y - (K @ x - 0.5 * x)).max() < 4 * n * 2.2e-16 * (np.abs(K) @ np.abs(x) + np.abs(x)).max()
    nys.close()


@pytest.mark.parametrize("panels", [256, 353])
def test_per_thread_stream(panels):
    import paper_2606_28865_amd as M
    n = 16 * panels
    print(f"case per-thread stream n={n}", flush=True)
    nys = M.Nystrom(3.0, _boundary(panels), stream=torch.cuda.ExternalStream(2))
    ref = M.Nystrom(3.0, _boundary(panels))
    x = torch.randn((2, 40, n), dtype=torch.float64, device="cuda")
    out = torch.empty_like(x)
    want = torch.stack([torch.stack([ref.apply(x[k, i], shift=-0.5) for i in range(40)]) for k in range(2)])
    torch.cuda.synchronize()

    def run(k):
        torch.cuda.set_device(0)
        for i in range(40):
            nys.apply(x[k, i], shift=-0.5, out=out[k, i])
        nys.stream.synchronize()                 # this thread's stream

    th = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert rel_err(out.cpu().numpy(), want.cpu().numpy()) < TOL
    nys.close()
    ref.close()
