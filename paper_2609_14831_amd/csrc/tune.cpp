// Autotuner for the forward graph pass: segment-to-wavefront tiling (long-target
// threshold, XCD remap), shared-triple tiles and quadratic-target blocks
// on/off, the B-chunk (sets per lane group) of the segment kernel, and
// optionally the choice between the two compensated float accumulation modes.
// Candidates are timed with HIP events on a private stream over zero-filled
// operands of the shape.
#include <algorithm>
#include <cstring>
#include <memory>
#include <utility>
#include <vector>

#include "internal.h"

using namespace cut;

namespace {

struct DevBuf {
    void* p = nullptr;
    explicit DevBuf(size_t bytes) {
        hipError_t e = hipMalloc(&p, bytes ? bytes : 1);
        if (e != hipSuccess) {
            p = nullptr;
            CUT_FAIL(CUT_E_NOMEM, "autotune: hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
        }
        HIP_CHECK(hipMemset(p, 0, bytes ? bytes : 1));
    }
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
};

double time_pass(Graph& g, int prec, int32_t nsets, int32_t nops, const void* eta, const void* x, double* y,
                 double* partials, size_t part_bytes, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    PassArgs p{};
    p.csr = &g.csr[0][0];
    p.A = eta;
    p.lda = nsets;
    p.B = x;
    p.ldb = (int64_t)nops * nsets;
    p.nsets = nsets;
    p.nops = nops;
    p.precision = prec;
    p.y = y;
    p.ldy = (int64_t)nops * nsets;
    p.scale = 1.0;
    p.part_bytes = part_bytes;
    for (int w = 0; w < 2; ++w) launch_forward(g, EPI_Y, p, partials, s);  // warm
    const int reps = 3;
    HIP_CHECK(hipEventRecord(e0, s));
    for (int r = 0; r < reps; ++r) launch_forward(g, EPI_Y, p, partials, s);
    HIP_CHECK(hipEventRecord(e1, s));
    HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    return ms / reps;
}

}  // namespace

extern "C" cut_status cut_graph_autotune(cut_graph_t h, int64_t nsets, int64_t nops, int32_t precision,
                                         int32_t allow_other_float, cut_tuning* out) {
    hipStream_t s = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    try {
        Graph& g = checked(h);
        check_prec(precision);
        check_shape(nsets, nops);
        if (!out) CUT_FAIL(CUT_E_INVAL, "cut_graph_autotune: null output");
        DeviceGuard dg(g.device);
        HIP_CHECK(hipDeviceSynchronize());
        const std::vector<int64_t> key = {nsets, nops, precision, allow_other_float};
        for (auto& kv : g.tune_cache)
            if (kv.first == key) {
                *out = kv.second;
                apply_tiling(g, out->long_records, out->chunk_records, out->tiling_flags);
                rereserve(g);
                return CUT_OK;
            }
        std::vector<int> precs = {precision};
        if (allow_other_float && precision == CUT_F32C) precs.push_back(CUT_F32X);
        if (allow_other_float && precision == CUT_F32X) precs.push_back(CUT_F32C);
        const size_t tb = precision == CUT_F64 ? 8 : 4;
        DevBuf eta(g.NG * nsets * tb), x(g.N * nsets * nops * tb), y(g.N * nsets * nops * 8);
        std::unique_ptr<DevBuf> part;
        size_t part_bytes = 0;
        // where every pass runs in triple space there is no tiling to choose, the
        // current one stays; a ragged flow's narrower passes may be on the records
        // where its full width is not, and take the tiling that is best for it
        const bool tiled = !triples_always(g, nsets, nops, precision);
        auto partials = [&](int pr) -> double* {
            const size_t need = tiled ? record_partial_bytes(g, (int32_t)nsets, (int32_t)nops, pr)
                                      : forward_partial_bytes(g, (int32_t)nsets, (int32_t)nops, pr);
            if (need == 0) return nullptr;
            if (!part || need > part_bytes) {
                part.reset();
                part.reset(new DevBuf(need));
                part_bytes = need;
            }
            return (double*)part->p;
        };
        HIP_CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        HIP_CHECK(hipEventCreate(&e0));
        HIP_CHECK(hipEventCreate(&e1));
        // Candidates (the graph's current tiling first) are timed round-robin
        // over 3 rounds and compared by their median, so clock drift during
        // tuning affects all of them alike; a candidate replaces the best only
        // when at least 2 % faster, so near-ties keep a stable choice.
        struct Cand {
            int64_t lr, cr;
            uint32_t flags;
            int prec;
            double ms[3];
        };
        std::vector<Cand> cands;
        cands.push_back({g.long_records, g.chunk_records, tiling_flags(g), precision, {0, 0, 0}});
        const int64_t lr = 1024;
        const int64_t crs[] = {64, 128, 256, 512};
        const uint32_t shapes[] = {0u, CUT_TILE_TRIPLE_CHUNKS, CUT_TILE_NO_CHUNKS, CUT_TILE_TRIPLES,
                                   CUT_TILE_QUAD_BLOCKS, CUT_TILE_QUAD_BLOCKS | CUT_TILE_TRIPLE_CHUNKS,
                                   CUT_TILE_QUAD_BLOCKS | CUT_TILE_TRIPLES};
        for (int64_t cr : crs)
            for (uint32_t xr = 0; tiled && xr <= 1; ++xr)
                for (uint32_t shape : shapes) {
                    if ((shape & CUT_TILE_TRIPLES) && !g.tiles.ok) continue;
                    if ((shape & CUT_TILE_TRIPLE_CHUNKS) && !g.triple_groups) continue;
                    if ((shape & CUT_TILE_QUAD_BLOCKS) && !g.qb.ok) continue;
                    // the chunk length does not change the unchunked, tile and block forms
                    if ((shape & (CUT_TILE_NO_CHUNKS | CUT_TILE_TRIPLES | CUT_TILE_QUAD_BLOCKS)) && cr != crs[3]) continue;
                    const uint32_t flags = (xr ? CUT_TILE_XCD_REMAP : 0u) | shape;
                    for (int pr : precs) cands.push_back({lr, cr, flags, pr, {0, 0, 0}});
                }
        auto time = [&](Cand& c, int round) {
            double* rows = partials(c.prec);
            // no bytes for products: the passes over the records
            c.ms[round] = time_pass(g, c.prec, (int32_t)nsets, (int32_t)nops, eta.p, x.p, (double*)y.p, rows,
                                    tiled ? 0 : part_bytes, s, e0, e1);
        };
        for (int round = 0; round < 3; ++round)
            for (Cand& c : cands) {
                apply_tiling(g, c.lr, c.cr, c.flags);
                time(c, round);
            }
        auto median = [](const double* v) { return std::max(std::min(v[0], v[1]), std::min(std::max(v[0], v[1]), v[2])); };
        const Cand& c0 = cands[0];
        cut_tuning best{c0.lr, c0.cr, c0.flags, c0.prec, median(c0.ms), median(c0.ms)};
        const double gain = 0.98;
        auto pick = [&](const std::vector<Cand>& cs, size_t from) {
            for (size_t i = from; i < cs.size(); ++i) {
                const double ms = median(cs[i].ms);
                if (ms < gain * best.pass_ms)
                    best = cut_tuning{cs[i].lr, cs[i].cr, cs[i].flags, cs[i].prec, ms, best.default_ms};
            }
        };
        pick(cands, 1);
        // second stage: the B-chunk (lane-group width) of the segment kernel,
        // on the three fastest tilings of the first stage, for every narrower
        // width the sets allow
        std::vector<size_t> order(cands.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(),
                         [&](size_t x, size_t y) { return median(cands[x].ms) < median(cands[y].ms); });
        std::vector<Cand> bc;
        int gw = 1;
        while (gw < nsets && gw < 64) gw <<= 1;
        for (size_t r = 0; tiled && r < std::min<size_t>(3, order.size()); ++r) {
            const Cand& c = cands[order[r]];
            const uint32_t base = c.flags & ~(3u << CUT_TILE_BCHUNK_SHIFT);
            for (uint32_t code = 1; code <= 3; ++code)
                if ((64 >> code) < gw)
                    bc.push_back({c.lr, c.cr, base | (code << CUT_TILE_BCHUNK_SHIFT), c.prec, {0, 0, 0}});
        }
        for (int round = 0; round < 3; ++round)
            for (Cand& c : bc) {
                apply_tiling(g, c.lr, c.cr, c.flags);
                time(c, round);
            }
        pick(bc, 0);
        apply_tiling(g, best.long_records, best.chunk_records, best.tiling_flags);
        rereserve(g);
        HIP_CHECK(hipEventDestroy(e0));
        HIP_CHECK(hipEventDestroy(e1));
        HIP_CHECK(hipStreamDestroy(s));
        g.tune_cache.push_back({key, best});
        *out = best;
        return CUT_OK;
    } catch (const Fail& f) {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (s) (void)hipStreamDestroy(s);
        return f.st;
    }
}
