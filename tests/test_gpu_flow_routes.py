"""Flows on each route of their passes over E_L (tests/flow_routes.py; the
launches themselves are checked there without a GPU): captured steps replay
bitwise as the stream path, twice; a flow resumed inside a repacked phase and a
checkpointed one, which keeps every set in its layout, are bitwise the same; and
against the oracle's RK4 with the tolerances of the other flow tests."""
import numpy as np
import pytest

import flow_routes as FR
import gpu_util as U
import workloads
from oracle import algebra as A
from oracle import native

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,nsets,nops,outside,prec,tiling,kernels", FR.RECORDS + FR.TRIPLES)
def test_flow_route(m, nsets, nops, outside, prec, tiling, kernels):
    from paper_2609_14831_amd import _lib as L
    U.say(f"[flow route] m {m} {nsets} x {nops} {prec} tiling {tiling}")
    g = U.outside_graph(L, m) if outside else U.graph(L, "majorana", m)
    P = getattr(L, "CUT_" + prec)
    z0 = workloads.small_majorana(m, nsets, nops, seed=m + nsets)
    ns = FR.steps(nsets)
    T = max(ns)

    def flow(flags, cuts=(), ckpt=0):
        z = torch.tensor(z0, device=DEV).contiguous()
        ck = torch.zeros(((T + 3) // 4,) + z0.shape, dtype=torch.float64, device=DEV) if ckpt else None
        ends = list(cuts) + [-1]
        for b, e in zip([0] + list(cuts), ends):
            p = L.flow_params(L.CUT_GEN_G2, P, 1e-2, 0.5, ckpt, flags=flags, step_begin=b, step_end=e)
            L.cut_flow_integrate(g, p, nsets, nops, ns, z, ck)
            torch.cuda.synchronize()
        return z.cpu().numpy()

    L.cut_graph_set_tiling(g, *tiling)
    try:
        a = flow(L.CUT_FLOW_HIPGRAPH)
        same = {"replayed again": flow(L.CUT_FLOW_HIPGRAPH), "stream order": flow(0),
                "resumed": flow(L.CUT_FLOW_HIPGRAPH, cuts=(T - 2,)), "checkpointed": flow(L.CUT_FLOW_HIPGRAPH, ckpt=4)}
    finally:
        L.cut_graph_set_tiling(g, 1024, 512, 0)
    for name, b in same.items():
        assert np.array_equal(a, b), name
    zr, _ = native.Engine(A.majorana_graph(m), "g2", 0.5).flow(z0, 1e-2, np.array(ns, dtype=np.int32))
    for s in range(nsets):
        for op in range(nops):
            d = np.linalg.norm(a[:, op, s] - zr[:, op, s]) / np.linalg.norm(zr[:, op, s])
            assert d < (1e-13 if prec == "F64" else 1e-7), (s, op, d)
