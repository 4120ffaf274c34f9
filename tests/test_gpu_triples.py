"""The triple-space contraction of Majorana graphs at the edges of its tiles:
one set, set blocks of 4, 8 and 16 and their remainders, pieces of the operand
columns, column tiles of 2, 4, 6, 8, 10, 14 and 16 modes (m = 14 .. 26); both
sides of the rule that chooses it; leading dimensions, accumulation, the
transposed actions and operands that are not finite, against the oracle.

Bounds: two FP64 summations of the same n terms in different orders differ by at
most 2 gamma_n S, S the sum of the terms' magnitudes (float operands: the
products are exact in FP64, so the same bound holds against the oracle on the
rounded operands).  CUT_F32C below the rule's line keeps the segment kernel's
compensated float sums and their bound.
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


_og = {}


def _graph(m):
    if m not in _og:
        og = A.graph_for("majorana", m)
        ga = A.Graph(og.algebra, og.size, og.N, og.k, og.i, og.j, np.abs(og.c), og.diag, og.pairs, og.gen_sign)
        _og[m] = (og, ga, U.sum_bound(int(np.diff(og.offsets()).max()) + 2))
    return _og[m]


def _padded(a, dt, pad):
    """Rows with `pad` trailing elements that must be neither read nor written."""
    buf = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), dtype=dt, device=DEV)
    buf[:, :a.shape[1]] = torch.tensor(a, device=DEV).to(dt)
    return buf[:, :a.shape[1]]


SIZES = [(12, 33), (14, 32), (14, 33), (14, 64), (14, 65), (16, 33), (18, 33), (20, 17), (22, 17), (24, 1), (24, 4),
         (24, 5), (26, 1), (26, 2), (26, 4), (26, 5), (26, 8), (26, 9), (26, 17)]
BELOW = [(12, 33), (14, 32), (20, 17), (22, 17), (24, 4), (24, 5)]  # float operands: the segment kernel


@pytest.mark.parametrize("prec", ["F64", "F32X", "F32C"])
@pytest.mark.parametrize("m,nsets", SIZES)
def test_apply_edges(L, m, nsets, prec):
    if prec == "F32C" and m == 26 and nsets > 5:
        pytest.skip("the launches of F32X")
    og, ga, bound = _graph(m)
    g = U.graph(L, "majorana", m)
    P = getattr(L, "CUT_" + prec)
    dt = torch.float64 if prec == "F64" else torch.float32
    for nops in ((1, 2, 3, 4, 5, 8) if (m, nsets) in ((14, 33), (26, 1)) else (3,) if m == 26 else (1, 3)):
        U.say(f"[triples] m {m} nsets {nsets} nops {nops} {prec}")
        eta = workloads.random_dense((og.N, nsets), seed=m + nsets, scale=0.5)
        x = workloads.random_dense((og.N, nops, nsets), seed=m + nsets + 1)
        y0 = workloads.random_dense((og.N, nops * nsets), seed=7)
        if prec != "F64":
            eta, x = U.f32(eta), U.f32(x)
        te, tx, ty = _padded(eta, dt, 3), _padded(x.reshape(og.N, -1), dt, 5), _padded(y0, torch.float64, 1)
        L.cut_graph_apply(g, 0, P, nsets, nops, te, tx, ty, L.CUT_ACCUMULATE)
        torch.cuda.synchronize()
        S = OGr.apply(ga, np.abs(eta), np.abs(x)).reshape(og.N, -1) + np.abs(y0)
        if prec == "F32C" and (m, nsets) in BELOW:
            bound = U.dot2_bound(int(np.diff(og.offsets()).max()) + 2)
        U.assert_within(ty.cpu().numpy(), y0 + OGr.apply(og, eta, x).reshape(og.N, -1), bound * S, "apply")
        assert bool(torch.isnan(ty._base[:, nops * nsets:]).all())


@pytest.mark.parametrize("prec", ["F64", "F32X"])
@pytest.mark.parametrize("m,nsets,nops", [(14, 32, 1), (14, 33, 2), (14, 65, 3), (26, 1, 1), (26, 1, 4), (26, 3, 2),
                                          (26, 8, 3), (26, 20, 2)])
def test_transposed_actions(L, m, nsets, nops, prec):
    """g_x and g_h of one action against the oracle's adjoints (the generator G2
    at the given h, its VJP from the oracle)."""
    from oracle import gen as OG
    og, ga, bound = _graph(m)
    g = U.graph(L, "majorana", m)
    h = workloads.random_dense((og.N, nsets), seed=1)
    x, w = (workloads.random_dense((og.N, nops, nsets), seed=s) for s in (2, 3))
    gen, vjp = OG.make_generator(og, "g2", 0.5)
    eta = gen(h)
    xr, wr = (x, w) if prec == "F64" else (U.f32(x), U.f32(w))
    er = eta if prec == "F64" else U.f32(eta)
    gx, gh = (torch.zeros((og.N, k), dtype=torch.float64, device=DEV) for k in (nops * nsets, nsets))
    t = lambda a: torch.tensor(a.reshape(og.N, -1), device=DEV)
    L.cut_graph_vjp(g, L.CUT_GEN_G2, 0.5, getattr(L, "CUT_" + prec), nsets, nops, t(h), t(x), t(w), gh, gx)
    torch.cuda.synchronize()
    ref = OGr.adjoint_x(og, er, wr)
    S = OGr.adjoint_x(ga, np.abs(er), np.abs(wr))
    # the generator's own rounding: a few FP64 operations on each eta
    U.assert_within(gx.cpu().numpy().reshape(ref.shape), ref, (bound + (1e-14 if prec == "F64" else 2 * U.U32)) * S + 1e-300, "g_x")
    geta = OGr.adjoint_eta(og, wr, xr)
    ref = vjp(h, geta)
    scale = np.abs(ref).max()
    assert np.abs(gh.cpu().numpy() - ref).max() <= 1e-12 * scale


@pytest.mark.parametrize("m,nsets,nops", [(14, 33, 1), (26, 1, 1), (26, 6, 2)])
@pytest.mark.parametrize("prec", ["F64", "F32C"])
def test_operands_that_are_not_finite(L, m, nsets, nops, prec):
    """An infinity or NaN reaches exactly the targets whose records touch it."""
    og, _, bound = _graph(m)
    g = U.graph(L, "majorana", m)
    P = getattr(L, "CUT_" + prec)
    dt = torch.float64 if prec == "F64" else torch.float32
    rng = np.random.default_rng(5)
    for bad in (np.inf, -np.inf, np.nan):
        for which in ("eta", "x"):
            eta = U.f32(workloads.random_dense((og.N, nsets), seed=11))
            x = U.f32(workloads.random_dense((og.N, nops, nsets), seed=12))
            for row in (3, 20, 44, 45, 101, og.N - 1):
                if which == "eta":
                    eta[row, rng.integers(nsets)] = bad
                else:
                    x[row, rng.integers(nops), rng.integers(nsets)] = bad
            y = torch.zeros((og.N, nops * nsets), dtype=torch.float64, device=DEV)
            L.cut_graph_apply(g, 0, P, nsets, nops, torch.tensor(eta, device=DEV).to(dt),
                              torch.tensor(x.reshape(og.N, -1), device=DEV).to(dt), y)
            with np.errstate(invalid="ignore"):
                ref = OGr.apply(og, eta, x).reshape(og.N, -1)
            got = y.cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(ref))
            inf = np.isinf(ref)
            assert np.array_equal(got[inf], ref[inf])
            fin = np.isfinite(ref)
            assert np.allclose(got[fin], ref[fin], rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("m,nsets", [(14, 33), (16, 40)])
def test_action_without_reservation(L, m, nsets):
    """No target of these graphs is split, so the records need no partial rows:
    an action on a handle that reserved nothing runs on them."""
    og, ga, bound = _graph(m)
    g = L.cut_graph_load(U.bundle_path(L, "majorana", m), 0, 0)
    try:
        eta = workloads.random_dense((og.N, nsets), seed=1)
        x = workloads.random_dense((og.N, 2, nsets), seed=2)
        y = torch.zeros((og.N, 2 * nsets), dtype=torch.float64, device=DEV)
        L.cut_graph_apply(g, 0, L.CUT_F64, nsets, 2, torch.tensor(eta, device=DEV),
                          torch.tensor(x.reshape(og.N, -1), device=DEV), y, reserve=False)
        torch.cuda.synchronize()
        S = OGr.apply(ga, np.abs(eta), np.abs(x)).reshape(og.N, -1)
        U.assert_within(y.cpu().numpy(), OGr.apply(og, eta, x).reshape(og.N, -1), bound * S, "apply")
        assert L.cut_graph_reserved_bytes(g) == 0
    finally:
        L.cut_graph_free(g)
