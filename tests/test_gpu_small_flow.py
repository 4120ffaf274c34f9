"""The one-launch flow of small graphs at its edges (targets per round, records
in LDS and beyond it, every operand count, finished sets, checkpoints, split
step ranges) against the launch-per-stage flow, which a timed call takes; and
the pair sums of the G2 generator's VJP at list lengths and set counts that are
no multiple of what a block covers, against the oracle.

Bounds: both flows sum the same terms in FP64 in different orders, so a step's
states differ by a few gamma_n of the terms' magnitudes; over these short flows
1e-12 of the norm.  With float operands a difference of one rounding enters a
stage as u32 of an element: 1e-7.
"""
import numpy as np
import pytest

import gpu_util as U
import workloads
from oracle import algebra as A
from oracle import gen as OG

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def L():
    from paper_2609_14831_amd import _lib
    return _lib


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("prec", ["F64", "F32X", "F32C"])
@pytest.mark.parametrize("alg,size,kind,nsets,nops", [
    ("epq", 2, "WEGNER_GRAPH", 1, 1), ("epq", 8, "WEGNER_GRAPH", 3, 2), ("epq", 9, "WEGNER_GRAPH", 1, 1),
    ("epq", 21, "WEGNER_GRAPH", 2, 1), ("majorana", 6, "G2", 2, 8), ("majorana", 8, "G2", 5, 1),
    ("majorana", 8, "WEGNER_GRAPH", 2, 6), ("majorana", 8, "G2", 33, 4), ("majorana", 10, "G2", 3, 3),
    ("majorana", 10, "G2", 1, 5), ("majorana", 10, "G2", 2, 7), ("majorana", 12, "G2", 32, 2),
    ("majorana", 12, "G2", 33, 2)])
def test_one_launch_flow(L, alg, size, kind, nsets, nops, prec):
    g = U.graph(L, alg, size)
    N = L.cut_graph_info(g)["n_ops"]
    U.say(f"[small flow] {alg} {size} {kind} {nsets} x {nops} {prec}")
    z0 = workloads.random_dense((N, nops, nsets), seed=size, scale=0.3)
    K, P = getattr(L, "CUT_GEN_" + kind), getattr(L, "CUT_" + prec)
    ns = [(5 * s) % 9 for s in range(nsets)]
    ns[-1] = 9
    C, T = 4, 9

    def flow(flags, **kw):
        z = torch.tensor(z0, device=DEV).contiguous()
        ck = torch.full(((T + C - 1) // C, N, nops, nsets), np.nan, dtype=torch.float64, device=DEV)
        for r in kw.get("ranges", [(0, -1)]):
            p = L.flow_params(K, P, 5e-3, 0.5, C, flags=flags, step_begin=r[0], step_end=r[1])
            L.cut_flow_integrate(g, p, nsets, nops, ns, z, ck)
        torch.cuda.synchronize()
        return z.cpu().numpy(), ck.cpu().numpy()

    z, ck = flow(0)
    zr, ckr = flow(L.CUT_FLOW_TIME_PASSES)
    tol = 1e-12 if prec == "F64" else 1e-7
    assert np.isfinite(z).all() and _rel(z, zr) <= tol and _rel(ck, ckr) <= tol
    zs, cks = flow(0, ranges=[(0, 3), (3, -1)])
    assert np.array_equal(z, zs) and np.array_equal(ck, cks)
    zh, ckh = flow(L.CUT_FLOW_HIPGRAPH)
    assert np.array_equal(z, zh) and np.array_equal(ck, ckh)
    for s in range(nsets):
        if ns[s] == 0:
            assert np.array_equal(z[:, :, s], z0[:, :, s])


@pytest.mark.parametrize("m", [6, 10, 16])
@pytest.mark.parametrize("nsets", [1, 3, 4, 5, 9])
def test_generator_vjp_pair_lists(L, m, nsets):
    og = A.majorana_graph(m)
    g = U.graph(L, "majorana", m)
    h = workloads.random_dense((og.N, nsets), seed=m)
    gb = workloads.random_dense((og.N, nsets), seed=m + 1)
    U.say(f"[g2 vjp] m {m} nsets {nsets}")
    _, vjp = OG.make_generator(og, "g2", 0.5)
    ref = vjp(h, gb)
    out = torch.zeros((og.N, nsets), dtype=torch.float64, device=DEV)
    L.cut_generator_vjp(g, L.CUT_GEN_G2, 0.5, nsets, torch.tensor(h, device=DEV), torch.tensor(gb, device=DEV), out)
    torch.cuda.synchronize()
    # the sums over a pair's list: gamma_n of their terms, n below N
    assert np.abs(out.cpu().numpy() - ref).max() <= U.sum_bound(og.N) * np.abs(ref).max() * 10
