"""Actions that may overlap on one handle: outside-space actions, and forward
actions whose passes over the records keep no partial rows, on two streams of
one handle at once.  Each result is bitwise that of the same call alone."""
import numpy as np
import pytest

import gpu_util as U
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def L():
    from paper_2609_14831_amd import _lib
    return _lib


@pytest.mark.parametrize("which,m,nsets,nops", [("outside", 20, 8, 3), ("flow", 14, 48, 2)])
def test_two_streams_of_one_handle(L, which, m, nsets, nops):
    g = U.outside_graph(L, m) if which == "outside" else U.graph(L, "majorana", m)
    w = L.CUT_GRAPH_OUTSIDE if which == "outside" else L.CUT_GRAPH_FLOW
    info = L.cut_graph_info(g)
    n, rows = info["n_ops"], info["n_out_ops"] if which == "outside" else info["n_ops"]
    t = lambda shape, seed: torch.tensor(workloads.random_dense(shape, seed=seed), device=DEV)
    ops = [(t((n, nsets), 3 * k), t((n, nsets * nops), 3 * k + 1)) for k in range(2)]
    ys = [torch.zeros((rows, nsets * nops), dtype=torch.float64, device=DEV) for _ in range(2)]
    alone = []
    for (eta, x), y in zip(ops, ys):
        L.cut_graph_apply(g, w, L.CUT_F64, nsets, nops, eta, x, y)
        torch.cuda.synchronize()
        alone.append(y.cpu().numpy().copy())
        y.fill_(float("nan"))
    assert np.isfinite(alone[0]).all() and not np.array_equal(alone[0], alone[1])
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rep in range(20):
        for k in ((0, 1), (1, 0))[rep % 2]:
            L.cut_graph_apply(g, w, L.CUT_F64, nsets, nops, *ops[k], ys[k], stream=streams[k].cuda_stream)
    torch.cuda.synchronize()
    for k in range(2):
        np.testing.assert_array_equal(ys[k].cpu().numpy(), alone[k])


@pytest.mark.parametrize("which,m,nsets,nops", [("outside", 20, 8, 2), ("flow", 14, 48, 1)])
def test_replays_beside_eager_calls(L, which, m, nsets, nops):
    """A captured action takes the records, which need no shared rows: replayed on one stream
    beside eager calls (products) on another, both are bitwise their results alone."""
    g = U.outside_graph(L, m) if which == "outside" else U.graph(L, "majorana", m)
    w = L.CUT_GRAPH_OUTSIDE if which == "outside" else L.CUT_GRAPH_FLOW
    info = L.cut_graph_info(g)
    n, rows = info["n_ops"], info["n_out_ops"] if which == "outside" else info["n_ops"]
    t = lambda shape, seed: torch.tensor(workloads.random_dense(shape, seed=seed), device=DEV)
    eta, x = t((n, nsets), 1), t((n, nsets * nops), 2)
    y, yc = (torch.zeros((rows, nsets * nops), dtype=torch.float64, device=DEV) for _ in range(2))
    call = lambda out, s: L.cut_graph_apply(g, w, L.CUT_F64, nsets, nops, eta, x, out, stream=s.cuda_stream, reserve=False)
    L.cut_graph_reserve(g, nsets, nops, 0, L.CUT_RESERVE_APPLY)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    call(y, a)
    torch.cuda.synchronize()
    alone = y.cpu().numpy().copy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=b):
        call(yc, b)
    graph.replay()
    torch.cuda.synchronize()
    captured = yc.cpu().numpy().copy()
    scale = np.abs(alone).max()
    assert np.abs(captured - alone).max() <= 1e-13 * scale and np.isfinite(captured).all()
    for rep in range(8):
        y.zero_()
        yc.zero_()
        torch.cuda.synchronize()
        call(y, a)
        with torch.cuda.stream(b):
            graph.replay()
        call(y, a)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), alone)
        np.testing.assert_array_equal(yc.cpu().numpy(), captured)
