"""cut_graph_apply_noalloc past its 64 MiB scratch: shapes whose partial rows in
triple space exceed it run in pieces of the operands or of the sets, bitwise the
result of cut_graph_apply (24 modes: 350 kB of partial rows a column)."""
import numpy as np
import pytest

import gpu_util as U
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("prec", ["F64", "F32C"])
@pytest.mark.parametrize("m,nsets,nops", [(24, 64, 8), (24, 200, 2), (24, 48, 4), (26, 1, 8)])
def test_pieces_are_bitwise_the_whole(m, nsets, nops, prec):
    from paper_2609_14831_amd import _lib as L
    g = U.graph(L, "majorana", m)
    n, P = L.cut_graph_info(g)["n_ops"], getattr(L, "CUT_" + prec)
    dt = torch.float64 if prec == "F64" else torch.float32
    U.say(f"[pieces] m {m} nsets {nsets} nops {nops} {prec}")
    eta = torch.tensor(workloads.random_dense((n, nsets), seed=1), device=DEV).to(dt)
    x = torch.tensor(workloads.random_dense((n, nsets * nops + 3), seed=2), device=DEV).to(dt)[:, :nsets * nops]
    y0, y1 = (torch.full((n, nsets * nops), 0.5, dtype=torch.float64, device=DEV) for _ in range(2))
    L.cut_graph_apply(g, 0, P, nsets, nops, eta, x, y0, L.CUT_ACCUMULATE)
    L.cut_graph_apply_noalloc(g, 0, P, nsets, nops, eta, x, y1, L.CUT_ACCUMULATE)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(y1.cpu().numpy(), y0.cpu().numpy())
