// Work-area reservation.  The computing entry points (actions, derivatives,
// flows) never allocate or synchronise: they carve their scratch out of work
// areas that only cut_graph_reserve and the tiling calls size.
#include <algorithm>

#include "internal.h"

namespace cut {

void* Workspace::need(size_t n, const char* what) const {
    if (n <= bytes) return ptr;
    CUT_FAIL(CUT_E_INVAL,
             "%s needs a work area of %zu bytes, %zu are reserved: call cut_graph_reserve with this shape "
             "(and again after a tiling change that adds partial rows)",
             what, n, bytes);
}

void Workspace::reserve(size_t n) {
    if (n <= bytes) return;
    if (ptr) {
        HIP_CHECK(hipDeviceSynchronize());
        (void)hipFree(ptr);
        ptr = nullptr;
        bytes = 0;
    }
    hipError_t e = hipMalloc(&ptr, n);
    if (e != hipSuccess) {
        ptr = nullptr;
        (void)hipGetLastError();  // reported here, not by a later call
        CUT_FAIL(CUT_E_NOMEM, "work area hipMalloc(%zu): %s", n, hipGetErrorString(e));
    }
    bytes = n;
}

void Workspace::reserve_optional(size_t n) {
    if (n <= bytes) return;
    size_t left = 0, total = 0;
    void* p = nullptr;
    if (hipMemGetInfo(&left, &total) != hipSuccess || n > left / 2 || hipMalloc(&p, n) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (ptr) {
        const hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) {
            (void)hipFree(p);
            CUT_FAIL(CUT_E_DEVICE, "hipDeviceSynchronize: %s", hipGetErrorString(e));
        }
        (void)hipFree(ptr);
    }
    ptr = p;
    bytes = n;
}

void Workspace::release() {
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
    bytes = 0;
}

// Bytes of partial rows in triple space for the layout and every smaller number
// of sets: fewer sets may be on the products' side of the line where more are not.
static size_t triples_reserve_bytes(const Graph& g, int64_t nsets, int64_t nops, int prec, bool transposed) {
    size_t b = triples_partial_bytes(g, nsets, nops, prec, transposed);
    for (int64_t n : {32, 16, 8, 4, 1})
        if (n < nsets) b = std::max(b, triples_partial_bytes(g, n, nops, prec, transposed));
    return b;
}

void reserve_shape(Graph& g, int64_t nsets, int64_t nops, int64_t ckpt_every, uint32_t what, bool extra) {
    size_t part = 0, tri = 0, outside = 0, small = 0, deriv = 0, ws = 0;
    bool area = false;  // whether the passes over the records keep partial rows
    for (int prec = CUT_F64; prec <= CUT_F32; ++prec) {
        const size_t rec = record_partial_bytes(g, (int32_t)nsets, (int32_t)nops, prec);
        area = area || rec > 0;
        if (what & (CUT_RESERVE_APPLY | CUT_RESERVE_DERIV)) part = std::max(part, rec);
        if (extra) tri = std::max(tri, triples_reserve_bytes(g, nsets, nops, prec, (what & (CUT_RESERVE_DERIV | CUT_RESERVE_ADJOINT)) != 0));
        if (what & CUT_RESERVE_DERIV)
            deriv = std::max({deriv, jvp_ws_bytes(g, nsets, nops, prec), vjp_ws_bytes(g, nsets, nops, prec)});
        if (what & CUT_RESERVE_FLOW)
            ws = std::max(ws, flow_ws_bytes(g, nsets, nops, prec, flow_outside_extra(g, nsets, nops)));
    }
    if (what & CUT_RESERVE_APPLY) {
        small = sizeof(double) * 2 * g.N * nsets;
        outside = outside_partial_bytes(g, nsets, nops);
    }
    if ((what & CUT_RESERVE_ADJOINT) && ckpt_every > 0)
        ws = std::max(ws, flow_ws_bytes(g, nsets, nops, CUT_F64, flow_adjoint_extra(g, nsets, nops, ckpt_every)));
    g.ws_part.reserve(part);
    g.ws_small.reserve(small);
    g.ws_deriv.reserve(deriv);
    g.ws.reserve(ws);
    if (!extra) return;
    // partial rows of products, in areas of their own (growing them moves none that
    // a captured pass over the records points into): without them the same calls run
    // on the records
    const bool apply = (what & CUT_RESERVE_APPLY) != 0;
    if (tri > 0 && ((apply && area) || (what & CUT_RESERVE_DERIV))) g.ws_prod.reserve_optional(std::max(part, tri));
    if (tri > 0 && (what & (CUT_RESERVE_FLOW | CUT_RESERVE_ADJOINT))) g.ws_tri.reserve_optional(std::max(part, tri));
    if (apply) g.rows.reserve_optional(std::max(outside, area ? 0 : tri));
}

void SharedRows::reserve_optional(size_t n) {
    std::lock_guard<std::mutex> lock(mu);
    if (n > 0 && !done) HIP_CHECK(hipEventCreateWithFlags(&done, hipEventDisableTiming));
    ws.reserve_optional(n);
}

SharedUse::SharedUse(SharedRows& r_, size_t least, hipStream_t s_) : r(r_), lock(r_.mu), s(s_) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (r.ws.bytes < least || !r.ws.ptr) return;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();  // the null stream while another stream is captured
        return;
    }
    if (st != hipStreamCaptureStatusNone) return;
    HIP_CHECK(hipStreamWaitEvent(s, r.done, 0));
    part = (double*)r.ws.ptr;
}

SharedUse::~SharedUse() {
    if (part) (void)hipEventRecord(r.done, s);
}

void SharedRows::release() {
    ws.release();
    if (done) (void)hipEventDestroy(done);
    done = nullptr;
}

void rereserve(Graph& g) {
    for (const auto& r : g.reserved) reserve_shape(g, r[0], r[1], r[2], (uint32_t)r[3], true);
}

}  // namespace cut

using namespace cut;

extern "C" cut_status cut_graph_reserve(cut_graph_t h, int64_t nsets, int64_t nops, int64_t ckpt_every,
                                        uint32_t what) {
    ABI_BEGIN
    Graph& g = checked(h);
    check_shape(nsets, nops);
    if (what == 0 || (what & ~15u)) CUT_FAIL(CUT_E_INVAL, "cut_graph_reserve: unknown flags 0x%x", what);
    if (ckpt_every < 0 || ((what & CUT_RESERVE_ADJOINT) && ckpt_every == 0))
        CUT_FAIL(CUT_E_INVAL, "cut_graph_reserve: CUT_RESERVE_ADJOINT needs ckpt_every > 0");
    DeviceGuard dg(g.device);
    // memory that was short for a shape is not asked for again on each call
    const std::vector<int64_t> key = {nsets, nops, ckpt_every, (int64_t)what};
    const bool known = std::find(g.reserved.begin(), g.reserved.end(), key) != g.reserved.end();
    reserve_shape(g, nsets, nops, ckpt_every, what, !known);
    if (!known) g.reserved.push_back(key);
    ABI_END
}

extern "C" cut_status cut_graph_reserved_bytes(cut_graph_t h, int64_t* bytes) {
    ABI_BEGIN
    Graph& g = checked(h);
    if (!bytes) CUT_FAIL(CUT_E_INVAL, "cut_graph_reserved_bytes: null output");
    *bytes = (int64_t)(g.ws.bytes + g.ws_small.bytes + g.ws_part.bytes + g.ws_prod.bytes + g.ws_tri.bytes + g.ws_deriv.bytes + g.rows.ws.bytes);
    ABI_END
}
