"""Results that are not finite, recomputed from the records by one lane, by 8 and by
a wavefront a target: one infinite operand in one set, in one column, in every
column, in all rows of a set, for quadratic and quartic rows; the infinities and
NaNs are exactly the oracle's and the other elements keep their bound."""
import numpy as np
import pytest

import gpu_util as U
import workloads
from oracle import algebra as A
from oracle import graph as OGr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("prec", ["F64", "F32X"])
@pytest.mark.parametrize("m,nsets,nops", [(26, 1, 1), (26, 5, 2), (26, 20, 2), (14, 40, 1)])
def test_recomputed_targets(m, nsets, nops, prec):
    from paper_2609_14831_amd import _lib as L
    og = A.graph_for("majorana", m)
    ga = A.Graph(og.algebra, og.size, og.N, og.k, og.i, og.j, np.abs(og.c), og.diag, og.pairs, og.gen_sign)
    bound = U.sum_bound(int(np.diff(og.offsets()).max()) + 2)
    g = U.graph(L, "majorana", m)
    dt = torch.float64 if prec == "F64" else torch.float32
    eta0 = U.f32(workloads.random_dense((og.N, nsets), seed=21))
    x0 = U.f32(workloads.random_dense((og.N, nops, nsets), seed=22))
    S = OGr.apply(ga, np.abs(eta0), np.abs(x0)).reshape(og.N, -1)
    cases = {"one quartic operand": (lambda e, x: x.__setitem__((og.N // 2, 0, nsets // 2), np.inf)),
             "one quadratic operand": (lambda e, x: x.__setitem__((7, nops - 1, 0), -np.inf)),
             "one row": (lambda e, x: x.__setitem__(og.N // 3, np.inf)),
             "one generator row": (lambda e, x: e.__setitem__(og.N - 5, -np.inf)),
             "one set": (lambda e, x: x.__setitem__((slice(None), slice(None), nsets - 1), np.nan))}
    for name, put in cases.items():
        U.say(f"[not finite] m {m} {nsets} x {nops} {prec} {name}")
        eta, x = eta0.copy(), x0.copy()
        put(eta, x)
        y = torch.zeros((og.N, nops * nsets), dtype=torch.float64, device=DEV)
        L.cut_graph_apply(g, 0, getattr(L, "CUT_" + prec), nsets, nops, torch.tensor(eta, device=DEV).to(dt),
                          torch.tensor(x.reshape(og.N, -1), device=DEV).to(dt), y)
        with np.errstate(invalid="ignore"):
            ref = OGr.apply(og, eta, x).reshape(og.N, -1)
        got = y.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(ref)), name
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        fin = np.isfinite(ref)
        if fin.any():
            U.assert_within(got[fin], ref[fin], (bound * S)[fin], name)
