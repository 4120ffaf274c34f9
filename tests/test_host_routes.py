"""Host side of the computing calls without a GPU (tests/fake_hip.cpp): which
kernels a call launches, in which order its streams are put, and what it
allocates."""
import pytest

import flow_routes as FR
import host_runtime as H


def _ordered(lines, streams, kernel):
    """Every use: a wait for the event that the use before it recorded after its last launch."""
    ev = {l.split()[2] for l in lines if l.split()[0] in ("wait", "record")}
    assert len(ev) == 1, lines
    want = []
    for s in streams:
        want += [("wait", s), ("kernel", s, kernel), ("kernel", s, "k_tri_combine"), ("record", s)]
    got = []
    for l in lines:
        w = l.split(" ", 3)
        got.append((w[0], w[1]) if w[0] != "kernel" else (w[0], w[1], w[3].split("<")[0]))
    assert got == want, lines


def test_outside_actions_on_two_streams_are_put_in_order():
    lines = H.run("""
g = graph(18, L.CUT_BUILD_OUTSIDE)
L.cut_graph_reserve(g, 8, 3, 0, L.CUT_RESERVE_APPLY)
log()
for s in (0x11, 0x22, 0x11):
    L.cut_graph_apply(g, 2, L.CUT_F64, 8, 3, Buf(8), Buf(24), Buf(24), stream=s)
out(log())
""")
    _ordered(lines, ["11", "22", "11"], "k_outside")


@pytest.mark.parametrize("tiling,m,nsets", [(0, 14, 33), (4, 24, 8)])   # no target split; CUT_TILE_NO_CHUNKS
def test_actions_without_partial_rows_on_two_streams_are_put_in_order(tiling, m, nsets):
    lines = H.run(f"""
g = graph({m})
L.cut_graph_set_tiling(g, 1 << 20, 512, {tiling})
L.cut_graph_reserve(g, {nsets}, 1, 0, L.CUT_RESERVE_APPLY)
log()
for s in (0x11, 0x22):
    L.cut_graph_apply(g, 0, L.CUT_F64, {nsets}, 1, Buf({nsets}), Buf({nsets}), Buf({nsets}), stream=s)
out(log())
""")
    _ordered(lines, ["11", "22"], "k_triples")


def test_area_of_overlapping_actions_is_not_the_chunked_passes_own():
    """An outside-space action may run beside a chunked pass: they share no partial rows."""
    out = H.run("""
g = graph(18, L.CUT_BUILD_OUTSIDE)
log()
L.cut_graph_reserve(g, 8, 3, 0, L.CUT_RESERVE_APPLY)
got = [int(l.split()[1]) for l in log() if l.startswith("malloc")]
out([got, L.cut_graph_reserved_bytes(g)])
""")
    sizes, total = out
    assert 4 * 18564 * 24 * 8 in sizes and len(sizes) == 3 and sum(sizes) == total


def test_captured_actions_without_partial_rows_run_on_the_records():
    out = H.run("""
g = graph(18, L.CUT_BUILD_OUTSIDE)
h = graph(14)
L.cut_graph_reserve(g, 8, 3, 0, L.CUT_RESERVE_APPLY)
L.cut_graph_reserve(h, 33, 1, 0, L.CUT_RESERVE_APPLY)
fake.fake_capturing(0x11, 1)
log()
L.cut_graph_apply(g, 2, L.CUT_F64, 8, 3, Buf(8), Buf(24), Buf(24), stream=0x11)
L.cut_graph_apply(h, 0, L.CUT_F64, 33, 1, Buf(33), Buf(33), Buf(33), stream=0x11)
out(log())
""")
    assert [l.split(" ", 3)[3].split("<")[0] for l in out] == ["k_pass", "k_pass"], out


@pytest.mark.parametrize("which,m,nsets", [(0, 14, 33), (2, 18, 8)])
def test_noalloc_leaves_the_scratch_alone_where_the_records_need_none(which, m, nsets):
    out = H.run(f"""
g = graph({m}, {"L.CUT_BUILD_OUTSIDE" if which else 0})
log()
L.cut_graph_apply_noalloc(g, {which}, L.CUT_F64, {nsets}, 1, Buf({nsets}), Buf({nsets}), Buf({nsets}), stream=0x11)
out(log())
""")
    assert [l.split(" ", 3)[3].split("<")[0] for l in out] == ["k_pass"], out


def _flow_passes(m, nsets, nops, steps, prec, tiling=None, outside=False):
    """The kernels over E_L (segment, chunk and triple-space passes) of a flow, in order."""
    lines = H.run(f"""
g = graph({m}, L.CUT_BUILD_OUTSIDE if {outside} else 0)
{"L.cut_graph_set_tiling(g, *" + repr(tiling) + ")" if tiling else ""}
L.cut_graph_reserve(g, {nsets}, {nops}, 0, L.CUT_RESERVE_FLOW)
log()
p = L.flow_params(L.CUT_GEN_G2, L.CUT_{prec}, 1e-3, flags=0, nonfinite=Buf(1))
steps = {steps}
L.cut_flow_integrate(g, p, {nsets}, {nops}, steps, Buf(1), stream=0x11, reserve=False)
out([k for k, _ in kernels(log())])
""")
    return [k for k in lines if k in ("k_pass", "k_triples", "k_triples1", "k_tile", "k_tile64", "k_qblock")]


def test_compacted_phases_take_the_route_of_the_full_layout():
    """24,800 FP64 columns are past the 2 GiB that 32-bit offsets reach: every pass runs on the
    records, also when the last 12 of the 3,100 sets are repacked into a layout of 16."""
    ks = _flow_passes(24, 3100, 8, "[3] * 12 + [1] * 3088", "F64")
    assert ks and set(ks) == {"k_pass"}, sorted(set(ks))
    # a layout within that reach, with as many sets left at the end: every pass in triple space
    ks = _flow_passes(24, 300, 8, "[3] * 12 + [1] * 288", "F64")
    assert ks and set(ks) == {"k_triples"}, sorted(set(ks))


@pytest.mark.parametrize("m,nsets,nops,launches", [(24, 8, 3, 1), (24, 64, 8, 4), (24, 200, 2, 2 * 2)])
def test_noalloc_takes_the_route_of_apply(m, nsets, nops, launches):
    """Past the scratch's 64 MiB (about 160 columns of 24 modes) the products run in pieces."""
    a, b = H.run(f"""
g = graph({m})
args = (g, 0, L.CUT_F64, {nsets}, {nops}, Buf({nsets}), Buf({nsets * nops}), Buf({nsets * nops}))
L.cut_graph_apply(*args, stream=0x11)
a = [k for k, _ in kernels(log())]
L.cut_graph_apply_noalloc(*args, stream=0x11)
out([a, [k for k, _ in kernels(log())]])
""")
    assert set(a) == set(b) == {"k_triples", "k_tri_combine"}
    assert b.count("k_triples") == launches


def test_optional_rows_that_do_not_fit_cost_nothing():
    """Short of memory for the outside-space partial rows of a larger shape: the reservation
    succeeds, areas held before stay, no error is left behind and later calls do not try again."""
    out = H.run("""
g = graph(18, L.CUT_BUILD_OUTSIDE)
L.cut_graph_reserve(g, 8, 3, 0, L.CUT_RESERVE_APPLY)
held = L.cut_graph_reserved_bytes(g)
fake.fake_limit(fake.fake_used() + (64 << 20))   # the larger shape's outside rows need 76 MiB
log()
L.cut_graph_reserve(g, 32, 4, 0, L.CUT_RESERVE_APPLY)
first = log()
L.cut_graph_reserve(g, 32, 4, 0, L.CUT_RESERVE_APPLY)
again = log()
a = lambda which, n, p: L.cut_graph_apply(g, which, L.CUT_F64, n, p, Buf(n), Buf(n * p), Buf(n * p), stream=0x11)
a(2, 8, 3), a(0, 8, 3), a(2, 32, 4)
out([held, L.cut_graph_reserved_bytes(g), first, again, [k for k, _ in kernels(log())]])
""")
    held, now, first, again, ks = out
    assert now >= held and again == []
    assert not any(l.startswith("free") and int(l.split()[1]) == 4 * 18564 * 24 * 8 for l in first)
    assert ks[:2] == ["k_outside", "k_tri_combine"]
    assert ks[-1] == "k_pass"   # the larger shape's action: not one of its operands fits


APPLY, FLOW, DERIV, ADJOINT = 1, 2, 4, 8


def _grown(m, nsets, nops, what):
    """Bytes that a reservation on a fresh handle adds."""
    return H.run(f"""
g = graph({m}, load=L.CUT_LOAD_ADJOINT)
L.cut_graph_reserve(g, {nsets}, {nops}, 4, {what})
out(L.cut_graph_reserved_bytes(g))
""")


@pytest.mark.parametrize("what", [APPLY, FLOW, DERIV, ADJOINT])
@pytest.mark.parametrize("m,nsets,nops", [(16, 32, 8), (22, 4, 5), (20, 40000, 3)])
def test_no_rows_are_reserved_for_products_that_cannot_run(m, nsets, nops, what):
    """Below the line at every width, or past the 2 GiB reach in every precision: no 4 N columns
    of doubles beside what the records and the state need."""
    n, cols = _strings(m), nsets * nops
    state = {APPLY: 2 * n * nsets,                                # generator-VJP scratch
             DERIV: n * (3 * nsets + 2 * cols),                   # generator, tangent and float shadows
             FLOW: n * (4 * cols + 2 * nsets),                    # two operands, accumulator, ordered state
             ADJOINT: n * ((4 + 17 + 4) * cols + 6 * nsets)}[what]
    chunks = 4 * m * m * cols                                    # partial rows of the quadratic targets
    assert _grown(m, nsets, nops, what) <= 8 * (state + chunks) * 1.05 + (1 << 20)


def _strings(m):
    return m * (m - 1) // 2 + m * (m - 1) * (m - 2) * (m - 3) // 24


@pytest.mark.parametrize("short", [False, True])
def test_products_give_way_where_their_rows_do_not_fit(short):
    """Memory for the records' passes and the state but not for the products' rows: every call
    that was reserved runs, on the records."""
    ks = H.run(f"""
g = graph(24, load=L.CUT_LOAD_ADJOINT)
n, s, o = 10902, 8, 3
if {short}:
    fake.fake_left(1 << 20)   # what the runtime reports as free
L.cut_graph_reserve(g, s, o, 0, L.CUT_RESERVE_APPLY)
L.cut_graph_reserve(g, s, o, 0, L.CUT_RESERVE_DERIV)
L.cut_graph_reserve(g, s, o, 0, L.CUT_RESERVE_FLOW)
log()
p = L.flow_params(L.CUT_GEN_G2, L.CUT_F64, 1e-3, flags=0, nonfinite=Buf(1))
L.cut_flow_integrate(g, p, s, o, [2] * s, Buf(1), stream=0x11, reserve=False)
L.cut_graph_apply(g, 0, L.CUT_F64, s, o, Buf(s), Buf(s * o), Buf(s * o), stream=0x11, reserve=False)
L.cut_graph_vjp(g, L.CUT_GEN_G2, 0.5, L.CUT_F64, s, o, Buf(s), Buf(s * o), Buf(s * o), Buf(s), Buf(s * o), stream=0x11,
                reserve=False)
out([k for k, _ in kernels(log())])
""")
    assert ("k_pass" in ks) == short and ("k_triples" in ks) == (not short)


@pytest.mark.parametrize("m,nsets,prec,tuned", [(24, 40, "F32X", True), (20, 24, "F64", True), (24, 24, "F64", False),
                                                (26, 40, "F32X", False)])
def test_autotune_where_narrower_passes_run_on_the_records(m, nsets, prec, tuned):
    """The full width runs in triple space in all four.  A ragged flow of the first two ends on the
    records (below 24 or 26 modes), so their tiling is chosen by timed passes over the records."""
    ks = H.run(f"""
g = graph({m})
log()
L.cut_graph_autotune(g, {nsets}, 3, L.CUT_{prec}, 0)
out([k for k, _ in kernels(log())])
""")
    assert ("k_triples" in ks) == (not tuned) and (ks.count("k_pass") > 40) == tuned
    steps = f"[4] * 2 + [1] * {nsets - 2}"
    flow = set(_flow_passes(m, nsets, 3, steps, prec))
    assert flow == ({"k_triples", "k_pass"} if tuned else {"k_triples"})


@pytest.mark.parametrize("threads", [0, 1])
def test_load_without_threads(threads):
    """The checks at load run in the calling thread where none can be started."""
    ks = H.run(f"""
import tempfile
with tempfile.TemporaryDirectory() as d:
    path = os.path.join(d, "g.cgb")
    L.cut_graph_build(L.CUT_ALG_MAJORANA, 26, path, 0, 0)
    fake.fake_threads({threads})
    g = L.cut_graph_load(path, 0, 0)
fake.fake_threads(-1)
L.cut_graph_apply(g, 0, L.CUT_F64, 4, 1, Buf(4), Buf(4), Buf(4), stream=0x11)
out([k for k, _ in kernels(log())])
""")
    assert ks == ["k_triples", "k_tri_combine"]


def test_load_where_the_products_tables_do_not_fit():
    """Short of memory at any of the tables' allocations the graph loads and runs on its records;
    nothing is lost."""
    out = H.run("""
import tempfile
with tempfile.TemporaryDirectory() as d:
    path = os.path.join(d, "g.cgb")
    L.cut_graph_build(L.CUT_ALG_MAJORANA, 20, path, 0, L.CUT_BUILD_OUTSIDE)
    log()
    g = L.cut_graph_load(path, 0, 0)
    used, before = 0, []   # bytes held before each allocation, and its size
    for l in log():
        if l.startswith("malloc"):
            before.append((used, int(l.split()[1])))
            used += before[-1][1]
        elif l.startswith("free"):
            used -= int(l.split()[1])
    L.cut_graph_free(g)
    res = []
    for held, size in before[-9:]:   # two tables, four of the outside space, three of its check
        fake.fake_limit(fake.fake_used() + held + size - 1)
        g = L.cut_graph_load(path, 0, 0)
        fake.fake_limit(288 << 30)
        log()
        for which in (0, 2):
            L.cut_graph_apply(g, which, L.CUT_F64, 20, 1, Buf(20), Buf(20), Buf(20), stream=0x11)
        res.append([k for k, _ in kernels(log())])
        L.cut_graph_free(g)
    out([res, fake.fake_used()])
""")
    res, left = out
    assert left == 0
    for k, ks in enumerate(res):
        assert ("k_triples" in ks) == (k >= 2) and "k_outside" not in ks, (k, ks)


@pytest.mark.parametrize("m,nsets,nops,outside,prec,tiling,kernels", FR.RECORDS + FR.TRIPLES + FR.SMALL)
def test_flows_run_the_kernels_they_are_tested_for(m, nsets, nops, outside, prec, tiling, kernels):
    ks = _flow_passes(m, nsets, nops, FR.steps(nsets), prec, tiling, outside)
    assert set(ks) == kernels, sorted(set(ks))


@pytest.mark.parametrize("m,nsets,prec,small", [(8, 2048, "F32X", True), (8, 2049, "F32X", False), (8, 2049, "F64", False),
                                                (12, 1536, "F32X", True), (12, 1537, "F32X", False),
                                                (10, 2049, "F32X", False), (10, 5000, "F64", True), (12, 5000, "F64", True)])
def test_one_launch_flows_up_to_the_sets_where_they_are_faster(m, nsets, prec, small):
    ks = H.run(f"""
g = graph({m})
L.cut_graph_reserve(g, {nsets}, 1, 0, L.CUT_RESERVE_FLOW)
log()
p = L.flow_params(L.CUT_GEN_G2, L.CUT_{prec}, 1e-3, flags=0, nonfinite=Buf(1))
L.cut_flow_integrate(g, p, {nsets}, 1, [2] * {nsets}, Buf(1), stream=0x11, reserve=False)
out([k for k, _ in kernels(log())])
""")
    assert ("k_flow_small" in ks) == small and ("k_pass" in ks) == (not small)


@pytest.mark.parametrize("m,nsets,nops,prec,flags,products", [
    # up to 32 sets
    (24, 1, 8, "F64", 0, True), (24, 4, 3, "F64", 0, False), (24, 8, 3, "F64", 0, True), (20, 17, 8, "F64", 0, True),
    (18, 17, 1, "F64", 0, False), (24, 16, 1, "F32X", 0, False), (24, 32, 5, "F32X", 0, True), (24, 32, 6, "F32X", 0, False),
    (24, 17, 4, "F32C", 0, True), (24, 17, 5, "F32C", 0, False), (26, 2, 8, "F32C", 0, True), (26, 32, 8, "F32C", 0, True),
    # above, default tiling
    (14, 33, 8, "F32C", 0, True), (18, 48, 8, "F32X", 0, True), (18, 49, 5, "F32X", 0, False), (18, 64, 4, "F32C", 0, True),
    (18, 65, 8, "F32X", 0, True), (18, 128, 5, "F32X", 0, False), (18, 64, 8, "F64", 0, True), (20, 64, 8, "F32C", 0, True),
    # above, B-chunk 32 or LDS tiles
    (14, 64, 1, "F64", 32, False), (14, 65, 1, "F64", 32, True), (14, 100, 2, "F32X", 32, False), (16, 48, 1, "F32X", 32, False),
    (16, 49, 8, "F32C", 32, True), (16, 33, 3, "F64", 2, True), (18, 100, 2, "F32C", 32, False), (18, 33, 8, "F64", 16, True),
    (20, 48, 4, "F32C", 32, True), (20, 48, 5, "F32C", 32, False), (20, 64, 1, "F32X", 2, False), (20, 65, 4, "F32X", 32, True),
    (22, 64, 5, "F32C", 32, True), (22, 64, 6, "F32C", 32, False), (22, 48, 8, "F32X", 32, True), (24, 64, 8, "F32C", 32, True),
])
def test_actions_take_products_on_their_side_of_the_line(m, nsets, nops, prec, flags, products):
    ks = H.run(f"""
g = graph({m})
L.cut_graph_set_tiling(g, 1024, 512, {flags})
log()
L.cut_graph_apply(g, 0, L.CUT_{prec}, {nsets}, {nops}, Buf({nsets}), Buf({nsets * nops}), Buf({nsets * nops}), stream=0x11)
out([k for k, _ in kernels(log())])
""")
    assert any(k.startswith("k_triples") for k in ks) == products, ks


def test_optional_rows_never_move_the_records_own():
    """Rows of products that become affordable later grow beside the area that passes over the
    records use, whose address a captured graph may hold."""
    out = H.run("""
g = graph(24)
fake.fake_left(1 << 20)
log()
L.cut_graph_reserve(g, 8, 3, 0, L.CUT_RESERVE_APPLY)
first = log()
fake.fake_left(1 << 40)
L.cut_graph_reserve(g, 8, 2, 0, L.CUT_RESERVE_APPLY)     # a smaller shape
out([first, log()])
""")
    first, later = out
    assert any(l.startswith("malloc") for l in first) and any(l.startswith("malloc") for l in later)
    assert not any(l.startswith("free") for l in later), later


@pytest.mark.parametrize("m,nsets,rows", [(18, 4, False), (18, 5, True), (20, 1, False), (20, 2, True)])
def test_outside_rows_only_where_the_products_can_run(m, nsets, rows):
    sizes, ks = H.run(f"""
g = graph({m}, L.CUT_BUILD_OUTSIDE)
log()
L.cut_graph_apply(g, 2, L.CUT_F64, {nsets}, 2, Buf({nsets}), Buf({2 * nsets}), Buf({2 * nsets}), stream=0x11)
lines = log()
out([[int(l.split()[1]) for l in lines if l.startswith("malloc")], [k for k, _ in kernels(lines)]])
""")
    n_out = {18: 18564, 20: 38760}[m]
    assert (4 * n_out * 2 * nsets * 8 in sizes) == rows and ("k_outside" in ks) == rows
