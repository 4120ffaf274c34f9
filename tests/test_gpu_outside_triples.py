"""The outside-space action of Majorana graphs as products over cuts into
triples, at the edges of its tiles (modes and pairs around the sizes of a row
and a column tile, set blocks of 4, 8 and 16, pieces of the operand columns):
against the oracle on sampled targets that hold every lowest mode, with leading
dimensions and accumulation; operands that are not finite; and a handle that
reserved no partial rows.

Bound: two FP64 summations of the same 20 (m - 6) terms in different orders
(float products are exact in FP64).
"""
import numpy as np
import pytest

import gpu_util as U
import workloads
from oracle import algebra as A
from oracle import graph as OGr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def L():
    from paper_2609_14831_amd import _lib
    return _lib


def _oracle(m, n_out):
    rows = np.unique(np.concatenate([np.linspace(0, n_out - 1, 24).astype(np.int64), [1, 2, n_out - 2]]))
    og = A.majorana_outside_graph(m, targets=rows)
    ga = A.OutsideGraph(m, og.N, og.n_out, og.k, og.i, og.j, np.abs(og.c), og.masks)
    return rows, og, ga


def _padded(a, dt, pad):
    buf = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), dtype=dt, device=DEV)
    buf[:, :a.shape[1]] = torch.tensor(a, device=DEV).to(dt)
    return buf[:, :a.shape[1]]


@pytest.mark.parametrize("prec", ["F64", "F32X", "F32C"])
@pytest.mark.parametrize("m,nsets,nops", [(16, 9, 1), (18, 4, 2), (18, 5, 2), (18, 8, 7), (18, 33, 5), (20, 1, 1),
                                          (20, 2, 6), (20, 4, 4), (20, 9, 3), (22, 1, 1), (22, 16, 1), (22, 17, 2),
                                          (24, 1, 3), (24, 3, 2)])
def test_outside_edges(L, m, nsets, nops, prec):
    g = U.outside_graph(L, m)
    n_out = L.cut_graph_info(g)["n_out_ops"]
    rows, og, ga = _oracle(m, n_out)
    P = getattr(L, "CUT_" + prec)
    dt = torch.float64 if prec == "F64" else torch.float32
    U.say(f"[outside triples] m {m} {nsets} x {nops} {prec}")
    eta = workloads.random_dense((og.N, nsets), seed=m, scale=0.5)
    x = workloads.random_dense((og.N, nops, nsets), seed=m + 1)
    if prec != "F64":
        eta, x = U.f32(eta), U.f32(x)
    ty = torch.full((n_out, nops * nsets + 1), float("nan"), dtype=torch.float64, device=DEV)
    ty[:, :-1] = 0.5
    L.cut_graph_apply(g, L.CUT_GRAPH_OUTSIDE, P, nsets, nops, _padded(eta, dt, 3), _padded(x.reshape(og.N, -1), dt, 5),
                      ty[:, :-1], L.CUT_ACCUMULATE)
    torch.cuda.synchronize()
    got = ty.cpu().numpy()
    assert np.isnan(got[:, -1]).all() and np.isfinite(got[:, :-1]).all()
    ref = OGr.apply_outside(og, eta, x)[rows].reshape(len(rows), -1)
    S = OGr.apply_outside(ga, np.abs(eta), np.abs(x))[rows].reshape(len(rows), -1) + 0.5
    # below the rule's line CUT_F32C keeps the compensated float sums
    below = prec == "F32C" and (m < 20 or (nsets == 1 and m < 22))
    bound = (U.dot2_bound if below else U.sum_bound)(20 * (m - 6) + 2)
    U.assert_within(got[rows, :-1], 0.5 + ref, bound * S, "outside")


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_outside_not_finite(L, bad):
    m, nsets, nops = 18, 5, 2
    g = U.outside_graph(L, m)
    og = A.majorana_outside_graph(m)
    eta = workloads.random_dense((og.N, nsets), seed=1)
    x = workloads.random_dense((og.N, nops, nsets), seed=2)
    eta[100, 1] = bad
    x[-1, 1, 3] = bad
    x[3, 0, 0] = bad  # a quadratic string: no outside record
    y = torch.zeros((og.n_out, nops * nsets), dtype=torch.float64, device=DEV)
    L.cut_graph_apply(g, L.CUT_GRAPH_OUTSIDE, L.CUT_F64, nsets, nops, torch.tensor(eta, device=DEV),
                      torch.tensor(x.reshape(og.N, -1), device=DEV), y)
    with np.errstate(invalid="ignore"):
        ref = OGr.apply_outside(og, eta, x).reshape(og.n_out, -1)
    got = y.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref)
    assert np.allclose(got[fin], ref[fin], rtol=1e-12, atol=1e-12)


def test_outside_without_reservation(L):
    m, nsets = 20, 3
    U.outside_graph(L, m)
    import os
    g = L.cut_graph_load(os.path.join(U._tmp, f"majorana_out_{m}.cgb"), 0, 0)
    try:
        n, n_out = L.cut_graph_info(g)["n_ops"], L.cut_graph_info(g)["n_out_ops"]
        eta = torch.tensor(workloads.random_dense((n, nsets), seed=1), device=DEV)
        x = torch.tensor(workloads.random_dense((n, nsets), seed=2), device=DEV)
        y, y2 = (torch.zeros((n_out, nsets), dtype=torch.float64, device=DEV) for _ in range(2))
        L.cut_graph_apply(g, L.CUT_GRAPH_OUTSIDE, L.CUT_F64, nsets, 1, eta, x, y, reserve=False)
        assert L.cut_graph_reserved_bytes(g) == 0
        L.cut_graph_apply(g, L.CUT_GRAPH_OUTSIDE, L.CUT_F64, nsets, 1, eta, x, y2)
        torch.cuda.synchronize()
        assert float((y - y2).abs().max()) <= 1e-13 * float(y.abs().max())
    finally:
        L.cut_graph_free(g)
