"""Flows and the kernels that their passes over E_L have to run, shared by the
tests on the GPU and the one that reads the launches without one."""

# (modes, sets, operands, built with E_C, precision, tiling, kernels of the passes)
# tilings: default; quadratic-target blocks with XCD remap (17); blocks and shared-triple
# tiles (19); tiles (2); triple chunks (8); B-chunk 16 with XCD remap (65)
RECORDS = [
    (14, 16, 2, False, "F32C", (1024, 512, 0), {"k_pass"}),
    (14, 16, 2, False, "F32C", (1024, 512, 17), {"k_pass", "k_qblock"}),
    (14, 16, 2, False, "F32C", (1024, 512, 19), {"k_pass", "k_qblock", "k_tile"}),
    (14, 16, 2, False, "F32X", (1024, 64, 8), {"k_pass"}),
    (14, 16, 2, False, "F64", (1024, 512, 2), {"k_pass", "k_tile"}),
    (14, 16, 2, False, "F32C", (1024, 512, 65), {"k_pass"}),
    (12, 40, 2, True, "F32C", (1024, 512, 0), {"k_pass"}),
    (12, 40, 2, True, "F32C", (1024, 512, 17), {"k_pass", "k_qblock"}),
    (12, 40, 2, True, "F32X", (1024, 512, 19), {"k_pass", "k_qblock", "k_tile64"}),
    (12, 40, 2, True, "F32C", (1024, 512, 65), {"k_pass"}),
    (22, 1, 1, False, "F64", (1024, 512, 0), {"k_pass"}),
    (22, 1, 1, False, "F32C", (64, 64, 1), {"k_pass"}),
    (22, 1, 1, False, "F64", (1024, 64, 8), {"k_pass"}),
]
# ragged: the active sets shrink through 16, 8, 4, 2 and 1
TRIPLES = [
    (26, 24, 2, False, "F64", (1024, 512, 0), {"k_triples"}),
    (26, 24, 2, False, "F32X", (1024, 512, 0), {"k_triples"}),
    (24, 1, 1, False, "F64", (1024, 512, 0), {"k_triples1"}),
]
SMALL = [(10, 4, 2, False, "F32C", (1024, 512, 0), set())]


def steps(nsets, most=12):
    """Ragged step counts from 2 to `most`: the first steps have every set active."""
    ns = [2 + (5 * s) % (most - 2) for s in range(nsets)]
    ns[nsets // 2] = most
    return ns
