// Triple-space contraction of the Majorana bracket: the plan built and checked
// at load, the combine of the partial rows with the pass's epilogue, and the
// launch (Sec. 2.2 Eq. graph-actions; Sec. 2.4 for the transposed uses).
//
// The plan is accepted only if the compiled records of E_L are exactly the
// records of the bracket in the kernels' form, factor by factor, so the
// contraction evaluates the compiled graph and nothing else.
//
// The bracket's structure constants c(k, i, j) are totally antisymmetric, so
// the transposed actions are brackets too:
//   sum_k,i c(k, i, j) e_i w_k = -L(e) w  at j,
//   sum_k,j c(k, i, j) w_k x_j =  L(x) w  at i.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <thread>
#include <unordered_map>
#include <vector>

#include "triples_kernel.h"

namespace cut {

void TriPlan::release_outside() {
    if (bin) (void)hipFree(bin);
    if (pair2) (void)hipFree(pair2);
    if (tri3) (void)hipFree(tri3);
    if (tasks) (void)hipFree(tasks);
    bin = pair2 = tri3 = nullptr;
    tasks = nullptr;
    out_ok = false;
}

void TriPlan::release() {
    release_outside();
    if (tab) (void)hipFree(tab);
    if (tmask) (void)hipFree(tmask);
    tab = nullptr;
    tmask = nullptr;
    ok = false;
}

static inline int above(uint64_t set, int q) { return __builtin_popcountll(set & ~((2ull << q) - 1)) & 1; }

// Sign of the record (target K; left I, right J) of the bracket in the form of
// the kernels, 0 when there is no such record.
static int record_sign(uint64_t K, uint64_t I, uint64_t J) {
    if ((I ^ J) != K) return 0;
    const int di = __builtin_popcountll(I), dj = __builtin_popcountll(J), dk = __builtin_popcountll(K);
    auto low = [](uint64_t x) { return __builtin_ctzll(x); };
    if (dk == 2 && di == dj && (di == 2 || di == 4)) {
        // t = I & J, one mode of K on each side: + sigma(t,u) sigma(t,v) when u (the lower) is on the left
        const uint64_t t = I & J;
        const int u = low(I & ~t), v = low(J & ~t);
        const int flip = (above(t, u) ^ above(t, v)) ^ (u < v ? 0 : 1);
        return flip ? -1 : 1;
    }
    if (dk == 4 && di + dj == 6 && (di == 2 || di == 4)) {
        const uint64_t Q = di == 2 ? I : J, F = di == 2 ? J : I;  // quadratic and quartic operand
        const uint64_t t = K & F;
        if (__builtin_popcountll(t) != 3) return 0;
        const int w = low(K & ~t), q = low(F & ~t);
        if (Q != ((1ull << w) | (1ull << q))) return 0;
        // generator quadratic: -, operand quadratic: +; times a2's sign (+ for w < q)
        const int flip = (above(t, w) ^ above(t, q)) ^ (w < q ? 0 : 1) ^ (di == 2 ? 1 : 0);
        return flip ? -1 : 1;
    }
    return 0;
}

// device copy of a host array in *dst, which its owner frees
template <class T>
static void upload(T** dst, const T* src, size_t count) {
    const hipError_t e = hipMalloc((void**)dst, count * sizeof(T));
    if (e != hipSuccess) {
        *dst = nullptr;
        (void)hipGetLastError();  // reported here, not by a later call
        CUT_FAIL(CUT_E_NOMEM, "hipMalloc(%zu bytes): %s", count * sizeof(T), hipGetErrorString(e));
    }
    HIP_CHECK(hipMemcpy(*dst, src, count * sizeof(T), hipMemcpyHostToDevice));
}

// modes below which no width is faster in triple space
constexpr int kTriMinModes = 14, kOutMinModes = 18;

void build_triples(Graph& g, const HostGraph& hg) {
    TriPlan& p = g.tri;
    p.release();
    const int m = hg.hdr.size;
    const int64_t N = hg.hdr.n_ops;
    if (hg.hdr.algebra != CUT_ALG_MAJORANA || m < kTriMinModes || m > 64 || hg.hdr.factor_bytes != 1) return;
    const int64_t nq = (int64_t)m * (m - 1) / 2, nt = nq * (m - 2) / 3, n4 = nt * (m - 3) / 4;
    if (N != nq + n4) return;
    const int64_t len2 = 2 * (m - 2) + (int64_t)(m - 2) * (m - 3) * (m - 4) / 3, len4 = 8 * (m - 4);
    std::unordered_map<uint64_t, int32_t> row;
    row.reserve((size_t)N * 2);
    const uint64_t all = m == 64 ? ~0ull : (1ull << m) - 1;
    for (int64_t k = 0; k < N; ++k) {
        const uint64_t L = hg.labels[k];
        if ((L & ~all) || __builtin_popcountll(L) != (k < nq ? 2 : 4)) return;
        if (!row.emplace(L, (int32_t)k).second) return;
    }
    // Every record has its sign and the common magnitude, no pair of inputs
    // comes twice in a target, and the target has as many as the bracket: the
    // two sets are the same.
    const int64_t* off = hg.off[0];
    const int32_t *ri = hg.ri[0], *rj = hg.rj[0];
    const int8_t* rc = hg.rc[0];
    if (off[1] == off[0]) return;
    const int c0 = rc[off[0]] * record_sign(hg.labels[0], hg.labels[ri[off[0]]], hg.labels[rj[off[0]]]);
    if (c0 == 0) return;
    std::atomic<bool> good{true};
    auto check = [&](int64_t k0, int64_t k1) {
        for (int64_t k = k0; k < k1 && good; ++k) {
            bool ok = off[k + 1] - off[k] == (k < nq ? len2 : len4);
            for (int64_t e = off[k]; ok && e < off[k + 1]; ++e) {
                ok = rc[e] == c0 * record_sign(hg.labels[k], hg.labels[ri[e]], hg.labels[rj[e]]);
                // stored in ascending (i, j) order, each pair once
                if (e > off[k] && (ri[e] < ri[e - 1] || (ri[e] == ri[e - 1] && rj[e] <= rj[e - 1]))) ok = false;
            }
            if (!ok) good = false;
        }
    };
    parallel_for(N, (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency())), check);
    if (!good) return;
    const int64_t ntau = nt + m;
    const int64_t ntp = ntau + 16;
    std::vector<uint32_t> tab((size_t)((m + 7) / 8 * 8 + 8) * ntp, kTriAbsent);
    std::vector<uint64_t> tau;
    for (int a = 0; a < m; ++a)
        for (int b = a + 1; b < m; ++b)
            for (int c = b + 1; c < m; ++c) tau.push_back((1ull << a) | (1ull << b) | (1ull << c));
    for (int a = 0; a < m; ++a) tau.push_back(1ull << a);
    for (int w = 0; w < m; ++w)
        for (int64_t t = 0; t < ntau; ++t) {
            if (tau[t] >> w & 1) continue;
            tab[(size_t)w * ntp + t] =
                (uint32_t)row.at(tau[t] | (1ull << w)) | (above(tau[t], w) ? kTriSign : 0u);
        }
    p.m = m;
    p.nq = (int32_t)nq;
    p.nt = (int32_t)nt;
    p.ntau = (int32_t)ntau;
    p.ntp = (int32_t)ntp;
    p.c = (double)c0;
    upload(&p.tab, tab.data(), tab.size());
    upload(&p.tmask, tau.data(), (size_t)nt);
    p.ok = true;
}

// ---------------------------------------------------------------- combine ----
struct TriCombineArgs {
    const double* p4;
    const double* p2;
    int32_t nstream, nq, nops, nsets, s0, w;  // sets [s0, s0 + w)
    int64_t N, ldp;
    double c;        // record factor, with the sign of a transposed use
    double scale;
    const int32_t* nsteps;
    const int32_t* step;
    double* y;
    int64_t ldy;
    int32_t accumulate;
    int32_t stage;
    double ds;
    double* z;
    double* acc;
    void* xout;
    int64_t ldx;
    double* hst;
    int64_t ldh;
    int32_t f32;
    // records and operands, for non-finite results
    const int64_t* off;
    const uint2* rec;
    const void* A;
    const void* B;
    int64_t lda, ldb;
    int32_t nred;
    double sign;
};

// The value of row `row` straight from its records (the kernels' zero padding
// gives NaN where an operand is not finite; the records have no such terms): the
// share of lane `lane` of LANES, which take records in turn, a few loaded before the
// first is used: where one operand is infinite nearly every quadratic target
// comes here.
template <int LANES>
__device__ __forceinline__ double tri_row(const TriCombineArgs& a, int64_t row, int op, int s, int lane) {
    constexpr int kBatch = 2;
    double v = 0.0;
    const int64_t end = a.off[row + 1];
    for (int64_t e = a.off[row] + lane; e < end && !__builtin_isnan(v); e += LANES * kBatch) {
        uint2 r[kBatch];
#pragma unroll
        for (int t = 0; t < kBatch; ++t) r[t] = a.rec[e + t * LANES < end ? e + t * LANES : e];
        for (int red = 0; red < a.nred; ++red) {
            const int64_t ca = (int64_t)red * a.nsets + s, cb = (int64_t)(red + op) * a.nsets + s;
            double x[kBatch], y[kBatch];
#pragma unroll
            for (int t = 0; t < kBatch; ++t) {
                const int64_t ia = (int64_t)(r[t].x & 0xFFFFFFu) * a.lda + ca, ib = (int64_t)(r[t].y & 0xFFFFFFu) * a.ldb + cb;
                x[t] = a.f32 ? (double)((const float*)a.A)[ia] : ((const double*)a.A)[ia];
                y[t] = a.f32 ? (double)((const float*)a.B)[ib] : ((const double*)a.B)[ib];
            }
#pragma unroll
            for (int t = 0; t < kBatch; ++t) {
                const double f = (double)__builtin_bit_cast(float, (r[t].x & 0xFF000000u) | ((r[t].y >> 24) << 16));
                if (e + t * LANES < end) v = __builtin_fma(f * x[t], y[t], v);
            }
        }
    }
    return a.sign * v;
}

template <int EPI>
__device__ __forceinline__ void tri_finish(const TriCombineArgs& a, int64_t row, int op, int s, double v) {
    const int64_t col = (int64_t)op * a.nsets + s;
    if constexpr (EPI == EPI_Y) {
        double& o = a.y[row * a.ldy + col];
        o = a.accumulate ? o + a.scale * v : a.scale * v;
    } else {
        const int64_t idx = row * a.ldx + col;
        const double nxt = rk_combine(a.stage, a.ds, a.z, a.acc, idx, v);
        if (a.f32) ((float*)a.xout)[idx] = (float)nxt;
        else ((double*)a.xout)[idx] = nxt;
        if (op == 0) a.hst[row * a.ldh + s] = nxt;
    }
}

// Partial rows of a target added in a fixed order, then the epilogue.  Blocks
// [0, nb2): 32 elements of the quadratic rows x 8 lanes over their streams
// (lane l adds streams l, l + 8, ..., then the lanes in order); the others: one
// thread per element of the quartic rows, its 4 slots in order.  Bound by the
// memory it streams (4 partial values per element and the epilogue's state):
// 0.29 ms at 40 modes x 320 columns, 0.94 GB of partial rows and 0.9 GB of state.
template <int EPI>
__global__ __launch_bounds__(256) void k_tri_combine(TriCombineArgs a, unsigned nb2) {
    __shared__ double red[8][32];
    const uint32_t cw = (uint32_t)a.nops * (uint32_t)a.w;
    if (blockIdx.x < nb2) {
        const uint64_t q = (uint64_t)blockIdx.x * 32 + threadIdx.x % 32;
        const int l = (int)threadIdx.x / 32;
        const bool in = q < (uint64_t)a.nq * cw;
        const int64_t row = in ? (int64_t)(q / cw) : 0;
        const uint32_t cc = in ? (uint32_t)(q % cw) : 0;
        const int op = (int)(cc / (uint32_t)a.w), s = a.s0 + (int)(cc % (uint32_t)a.w);
        const bool act = in && (a.nsteps == nullptr || a.nsteps[s] > *a.step);
        double v = 0.0;
        if (act) {
            const double* p = a.p2 + row * a.ldp + (int64_t)op * a.nsets + s;
            for (int r = l; r < a.nstream; r += 8) v += __builtin_nontemporal_load(p + (int64_t)r * a.nq * a.ldp);
        }
        const int el = (int)threadIdx.x % 32, lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x / 64;
        red[l][el] = v;
        __syncthreads();
        v = red[0][el];
        for (int k = 1; k < 8; ++k) v += red[k][el];
        v *= a.c;
        const bool odd = act && !__builtin_isfinite(v);
        if (l == 0 && act && !odd) tri_finish<EPI>(a, row, op, s, v);
        // Every wavefront knows the block's non-finite elements (the same sums of the
        // same 32).  Many sets of a row: 8 lanes to each, whose loads share lines; else
        // the wavefronts take them in turn, 64 lanes to each.  An action of 40 modes
        // with one infinite operand, one lane a target -> this, ms (on the records):
        // 64 x 5 in one set 13.4 -> 1.5 (3.5), in every column 15.8 -> 3.1; 1 x 1 5.9 -> 0.8 (0.18).
        uint32_t todo = (uint32_t)__ballot(odd);
        if (__popc(todo) > 8 && a.w > 8) {
            __syncthreads();
            red[l][el] = odd ? tri_row<8>(a, row, op, s, l) : 0.0;
            __syncthreads();
            if (l != 0 || !odd) return;
            v = red[0][el];
            for (int k = 1; k < 8; ++k) v += red[k][el];
            tri_finish<EPI>(a, row, op, s, v);
            return;
        }
        for (int n = 0; todo; ++n, todo &= todo - 1) {
            if ((n & 3) != wave) continue;
            const int from = __ffs((int)todo) - 1;
            const int64_t r = __shfl((int)row, from);
            const int o = __shfl(op, from), t = __shfl(s, from);
            double p = tri_row<64>(a, r, o, t, lane);
            for (int d = 1; d < 64; d <<= 1) p += __shfl_xor(p, d);
            if (lane == 0) tri_finish<EPI>(a, r, o, t, p);
        }
        return;
    }
    const uint64_t q = (uint64_t)(blockIdx.x - nb2) * 256 + threadIdx.x;
    if (q >= (uint64_t)(a.N - a.nq) * cw) return;
    uint64_t r4;
    uint32_t cc;
    if (q < (1ull << 32)) {
        r4 = (uint32_t)q / cw;
        cc = (uint32_t)q - (uint32_t)r4 * cw;
    } else {
        r4 = q / cw;
        cc = (uint32_t)(q % cw);
    }
    const int64_t row = a.nq + (int64_t)r4;
    const int op = (int)(cc / (uint32_t)a.w), s = a.s0 + (int)(cc % (uint32_t)a.w);
    if (a.nsteps && a.nsteps[s] <= *a.step) return;
    const double* p = a.p4 + row * a.ldp + (int64_t)op * a.nsets + s;
    const int64_t st = a.N * a.ldp;
    double v = a.c * (((__builtin_nontemporal_load(p) + __builtin_nontemporal_load(p + st)) +
                       __builtin_nontemporal_load(p + 2 * st)) +
                      __builtin_nontemporal_load(p + 3 * st));
    if (__builtin_expect(!__builtin_isfinite(v), 0)) v = tri_row<1>(a, row, op, s, 0);
    tri_finish<EPI>(a, row, op, s, v);
}

// ----------------------------------------------------------------- launch ----
// Shape of a launch over w sets: set quads per block (0: the one-set kernel),
// blocks of sets, and streams of the quadratic blocks.  Everything that decides
// the order of a sum is a function of the plan and w.
struct TriShape {
    int sq, chunks, tw, nwt, nbp, nstream;
};

static TriShape tri_shape(const TriPlan& p, int w) {
    TriShape t;
    t.sq = w <= 1 ? 0 : w <= 4 ? 1 : w <= 8 ? 2 : 4;
    t.chunks = t.sq == 4 ? (w + 15) / 16 : 1;
    t.tw = t.sq ? 4 / t.sq : 1;
    // column tiles: 16 modes, 8 in the one-set kernel; tile pairs u <= v of 16
    // rows (tw of them to a block) and one column tile
    t.nwt = t.sq ? (p.m + 15) / 16 : (p.m + 7) / 8;
    t.nbp = 0;
    for (int v = 0; v < t.nwt; ++v) t.nbp += (t.sq ? v / t.tw : v / 2) + 1;
    const int steps = t.sq ? (p.ntau + 3) / 4 : (p.ntau + 15) / 16;
    if (t.sq == 0) {
        // about 1024 wavefronts of at least 4 steps
        t.nstream = std::max(1, std::min(1024 / t.nbp, steps / 4));
    } else {
        // 512 blocks are resident (two per CU).  The quadratic ones start first
        // and the quartic ones fill in behind: half of the places for one block
        // of sets, more with several; where quartic and quadratic blocks together
        // can all be resident without streams much longer than a quartic
        // block, what the quartic ones leave.  Streams of fewer than 8 steps are
        // mostly their first loads.  A step, 5 FP64 operands, us, 512 places
        // in every case -> this: 24 modes x 16 sets 393 -> 305, 28 x 8 404 -> 300,
        // 32 x 8 547 -> 409, 26 x 16 473 -> 379, 36 x 3 559 -> 510, 32 x 32 1300 -> 1272;
        // 24 x 32 519 -> 541.
        const int q4 = (p.nt + 16 * t.tw - 1) / (16 * t.tw) * t.nwt;
        int places = t.chunks == 1 ? 256 : t.chunks == 2 ? 320 : 512;
        const int left = 512 - q4;
        if (t.chunks == 1 && left > 0 && left < places) {
            if (steps * t.nbp <= 24 * left) places = left;
            else if (t.sq == 4) places = 512;  // a second round either way: short streams
        }
        t.nstream = std::max(1, std::min(places / (t.nbp * t.chunks), steps / 8));
    }
    if (t.nstream >= 8) t.nstream &= ~7;  // whole streams per XCD
    return t;
}

// partial rows of one column, for the most streams of any width
static size_t tri_column_bytes(const Graph& g) {
    int streams = 1;
    for (int w : {1, 4, 8, 16, 32, 48}) streams = std::max(streams, tri_shape(g.tri, w).nstream);
    return (size_t)(4 * g.N + (int64_t)streams * g.tri.nq) * sizeof(double);
}


// Sets that decide a launch's shape: as wide as the segment kernel's lane
// groups, at least min(8, nsets).
static int tri_width(const PassArgs& a) {
    const int w = a.s1 > 0 ? a.s1 - a.s0 : a.nsets;
    return std::max({w, std::min(8, (int)a.nsets), (int)a.gfloor});
}

// Whether the rows of a layout of ld elements a row are within reach of the
// kernels' 32-bit byte offsets.
static bool tri_reach(const Graph& g, int64_t ld, bool f64) { return g.N * ld * (f64 ? 8 : 4) < (int64_t)0x7FFFFFFF; }

// FP64 and the compensated float modes (the sums are FP64 with exact products,
// at least as accurate as either); 32-bit offsets into both operand arrays.
// Every launch costs a fixed latency (two kernels, at least m / 4 dependent
// steps of 1.6 us), which the records' E x columns have to outweigh.  Up to 32
// sets the segment kernel's lanes are full and it is best at float with 2 to 16
// sets; above, its groups of 64 lanes are worst just past 32 and 64 sets, unless
// the tiling gives it narrower groups or stages rows in LDS (`tuned`, what
// cut_graph_autotune finds there).  The products run whole blocks of 16 sets and
// column tiles of 16 modes, so 16 modes are better for them than 18.  One action,
// us, records -> products (F: F32X, C: F32C):
//   up to 32 sets, modes x sets x operands
//     above the line  24x1x3 FP64 25 -> 17;  24x8x3 FP64 53 -> 29;  20x17x3 FP64 68 -> 32
//                     26x2x2 F 30 -> 20;  26x8x8 C 81 -> 77;  24x17x4 C 74 -> 64;  24x32x5 F 93 -> 88
//     below it        18x8x3 C 11 -> 20;  20x4x3 FP64 16 -> 24;  22x16x5 C 36 -> 47;  24x24x8 C 125 -> 137
//                     (but 22x16x3 FP64 59 -> 37 and 24x8x3 C 32 -> 26: products of 24 modes with 2
//                     to 16 float sets are 1.06 to 1.5 times faster, of 22 with 8 or 16 FP64 sets
//                     1.04 to 1.7, of 16 with 17 to 32 FP64 sets 1.5 to 1.9)
//   above 32, default tiling
//     above the line  14x33x3 FP64 62 -> 32, F 41 -> 26;  14x64x6 F 1.09, 18x33x8 C 1.36, 18x64x4 F 1.04 times
//     below it        18x64x6 F 78 -> 86;  18x128x6 F 111 -> 132
//   above 32, tuned
//     above the line  14x100x4 FP64 1.28, 16x33x1 FP64 1.46, 18x48x5 FP64 1.06, 16x49x8 C 1.05,
//                     20x48x2 C 1.01, 20x128x4 C 1.01, 22x64x5 C 1.02 times
//     below it        14x48x8 C 25 -> 57, 14x33x4 FP64 0.66, 16x48x8 C 0.85, 18x64x5 C 0.56,
//                     20x64x5 F 0.89, 22x64x8 C 0.96 of its speed
// The transposed actions' passes over the records have neither chunks nor narrow
// groups: the line of the default tiling, for any number of operands (a VJP of 2
// FP64 operands 1.1 to 4.8 times faster wherever it is taken).
static bool tri_faster(const Graph& g, int w, int64_t nops, int32_t precision, bool transposed) {
    const int m = g.tri.m;
    const bool f64 = precision == CUT_F64;
    if (w <= 32) {
        int least = f64 && w > 16 ? 20 : w == 1 || w > (f64 ? 4 : 16) ? 24 : 26;
        if (!f64 && w > 16 && !transposed && nops > (precision == CUT_F32C ? 4 : 5)) least = 26;
        return m >= least;
    }
    if (transposed) return m >= kTriMinModes;
    const bool tuned = g.bchunk != 0 || g.use_tiles || g.use_quadblocks;
    const int last = (w - 1) % 64 + 1;  // sets in the last group of 64 lanes
    if (!tuned) return m >= kTriMinModes && (f64 || m != 18 || nops <= 4 || last <= (w > 64 ? 32 : 48));
    if (f64) return m >= 16 || w > 64;
    if (m >= 22) return m > 22 || nops <= 5 || w <= 48 || w > 64;
    return m == 20 ? nops <= 4 && (w <= 48 || w > 64) : m == 16 && w > 48;
}

// fn(w) for a width of each kind on either side of the line among those of the
// passes over a layout (min(8, nsets) to nsets)
template <class F>
static bool tri_any_width(int64_t nsets, F fn) {
    const int64_t lo = std::min<int64_t>(8, nsets);
    for (int64_t w : {lo, (int64_t)17, (int64_t)33, (int64_t)49, (int64_t)65, nsets})
        if (w >= lo && w <= nsets && fn((int)w)) return true;
    return false;
}

size_t triples_partial_bytes(const Graph& g, int64_t nsets, int64_t nops, int32_t precision, bool transposed) {
    if (!g.tri.ok || precision == CUT_F32 || !tri_reach(g, nops * nsets, precision == CUT_F64)) return 0;
    const bool any = tri_any_width(nsets, [&](int w) {
        return tri_faster(g, w, nops, precision, false) || (transposed && tri_faster(g, w, nops, precision, true));
    });
    return any ? tri_column_bytes(g) * (size_t)(nops * nsets) : 0;
}

bool triples_always(const Graph& g, int64_t nsets, int64_t nops, int32_t precision) {
    if (!g.tri.ok || precision == CUT_F32 || !tri_reach(g, nops * nsets, precision == CUT_F64)) return false;
    return !tri_any_width(nsets, [&](int w) { return !tri_faster(g, w, nops, precision, false); });
}

bool triples_usable(const Graph& g, const PassArgs& a) {
    if (!g.tri.ok || a.precision == CUT_F32) return false;
    const bool transposed = a.csr != &g.csr[0][0];
    if (!tri_faster(g, tri_width(a), a.nops, a.precision, transposed)) return false;
    if (!tri_reach(g, std::max({a.lda, a.ldb, a.ldfull}), a.precision == CUT_F64)) return false;
    return a.part_bytes >= tri_column_bytes(g) * (size_t)((int64_t)a.nops * a.nsets);
}

void launch_triples(const Graph& g, int epi, const PassArgs& a, int nred, double sign, double* part, hipStream_t s) {
    const TriPlan& p = g.tri;
    const bool f32 = a.precision != CUT_F64;
    const int s0 = a.s1 > 0 ? a.s0 : 0, s1 = a.s1 > 0 ? a.s1 : a.nsets;
    const TriShape sh = tri_shape(p, tri_width(a));
    const int64_t esz = f32 ? 4 : 8;
    TriArgs t{};
    t.tab = p.tab;
    t.tmask = p.tmask;
    t.m = p.m;
    t.nt = p.nt;
    t.ntau = p.ntau;
    t.ntp = p.ntp;
    t.nq = p.nq;
    t.N = g.N;
    t.lda = (int32_t)a.lda;
    t.ldb = (int32_t)a.ldb;
    t.nsets = a.nsets;
    t.s0 = s0;
    t.s1 = s1;
    t.nred = nred;
    t.nsteps = a.nsteps;
    t.step = a.step;
    t.ldp = (int64_t)a.nops * a.nsets;
    t.nbp = sh.nbp;
    t.nstream = sh.nstream;
    t.nwt = sh.nwt;
    // columns of the arrays: the generator side has nred column blocks, the
    // operand side nops (nred of them in a transposed use)
    const int64_t bytesA = ((g.N - 1) * a.lda + (int64_t)nred * a.nsets) * esz;
    const int64_t bytesB = ((g.N - 1) * a.ldb + (int64_t)std::max((int)a.nops, nred) * a.nsets) * esz;
    double* p4 = part;
    double* p2 = part + 4 * g.N * t.ldp;
    const int most = f32 ? tri_ops<float>() : tri_ops<double>();
    for (int o = 0; o < a.nops;) {
        const int left = a.nops - o, pieces = (left + most - 1) / most, n = (left + pieces - 1) / pieces;
        const int64_t bo = (int64_t)o * a.nsets * esz;
        t.A = a.A;
        t.B = (const char*)a.B + bo;
        t.bytesA = (uint32_t)bytesA;
        t.bytesB = (uint32_t)(bytesB - bo);
        t.p4 = p4 + (int64_t)o * a.nsets;
        t.p2 = p2 + (int64_t)o * a.nsets;
        // twice the triples per wavefront where that still leaves 4 blocks per CU
        auto tiles = [&](int ti) { return (p.nt + 4 * ti * sh.tw - 1) / (4 * ti * sh.tw); };
        const int ti = tri_rows(n, (int)esz) == 8 && sh.sq == 4 && (int64_t)tiles(8) * t.nwt * sh.chunks >= 1024 ? 8 : 4;
        t.ntt = tiles(ti);
        t.per = (t.ntt + 7) / 8;
        dim3 grid;
        if (sh.sq == 0) {
            t.nb2 = t.nbp * t.nstream;
            grid = dim3((unsigned)((t.nb2 + t.ntt * t.nwt + 3) / 4));
        } else {
            t.chunks = (s1 - s0 + 4 * sh.sq - 1) / (4 * sh.sq);
            t.nb2 = t.nbp * ((t.nstream + 7) / 8) * 8 * t.chunks;
            grid = dim3((unsigned)(t.nb2 + 8 * t.per * t.nwt * t.chunks));
        }
        if (f32) launch_triples_t<float>(t, n, sh.sq, ti, grid, s);
        else launch_triples_t<double>(t, n, sh.sq, ti, grid, s);
        o += n;
    }
    TriCombineArgs c{};
    c.p4 = p4;
    c.p2 = p2;
    c.nstream = sh.nstream;
    c.nq = p.nq;
    c.nops = a.nops;
    c.nsets = a.nsets;
    c.s0 = s0;
    c.w = s1 - s0;
    c.N = g.N;
    c.ldp = t.ldp;
    c.c = p.c * sign;
    c.scale = a.scale;
    c.nsteps = a.nsteps;
    c.step = a.step;
    c.y = (double*)a.y;
    c.ldy = a.ldy;
    c.accumulate = a.accumulate;
    c.stage = a.stage;
    c.ds = a.ds;
    c.z = a.z;
    c.acc = a.acc;
    c.xout = a.xout;
    c.ldx = a.ldb;
    c.hst = a.hst;
    c.ldh = a.ldh;
    c.f32 = f32 ? 1 : 0;
    c.off = g.csr[0][0].off;
    c.rec = g.csr[0][0].rec;
    c.A = a.A;
    c.B = a.B;
    c.lda = a.lda;
    c.ldb = a.ldb;
    c.nred = nred;
    c.sign = sign;
    const int64_t cw = (int64_t)a.nops * c.w;
    const unsigned nb2 = (unsigned)((p.nq * cw + 31) / 32);
    const unsigned nb = nb2 + (unsigned)(((g.N - p.nq) * cw + 255) / 256);
    if (epi == EPI_Y) hipLaunchKernelGGL((k_tri_combine<EPI_Y>), dim3(nb), dim3(256), 0, s, c, nb2);
    else hipLaunchKernelGGL((k_tri_combine<EPI_RK>), dim3(nb), dim3(256), 0, s, c, nb2);
}

void launch_triples_in(const Graph& g, const PassArgs& a, double* part, size_t bytes, hipStream_t s) {
    // whole operands while their columns fit, else ranges of the sets of one;
    // every piece has the shape of the whole launch (its width), so each sum is
    // bitwise the whole launch's
    const int64_t fit = (int64_t)(bytes / tri_column_bytes(g)), esz = a.precision == CUT_F64 ? 8 : 4;
    if (fit < 1) CUT_FAIL(CUT_E_INVAL, "partial rows of one column need %zu bytes, there are %zu", tri_column_bytes(g), bytes);
    int64_t ops = std::max<int64_t>(1, std::min<int64_t>(a.nops, fit / a.nsets)), sets = std::min<int64_t>(a.nsets, fit);
    if (sets < a.nsets && sets > 16) sets &= ~15;  // whole blocks of sets
    for (int64_t o = 0; o < a.nops; o += ops)
        for (int64_t s0 = 0; s0 < a.nsets; s0 += sets) {
            const int64_t b = o * a.nsets + s0;
            PassArgs q = a;
            q.gfloor = tri_width(a);
            q.nops = (int32_t)std::min<int64_t>(ops, a.nops - o);
            q.nsets = (int32_t)std::min<int64_t>(sets, a.nsets - s0);
            q.A = (const char*)a.A + s0 * esz;
            q.B = (const char*)a.B + b * esz;
            q.y = (double*)a.y + b;
            launch_triples(g, EPI_Y, q, 1, 1.0, part, s);
        }
}

void launch_adjoint_x(const Graph& g, const PassArgs& a, double* part, hipStream_t s) {
    if (part && triples_usable(g, a)) launch_triples(g, EPI_Y, a, 1, -1.0, part, s);
    else launch_pass(MODE_BCAST, EPI_Y, a, s);
}

// out_i = sum_op L(x_op) w_op: the operand takes the generator's place and the
// cotangent the operand's
void launch_adjoint_eta(const Graph& g, const PassArgs& a, double* part, hipStream_t s) {
    if (part && triples_usable(g, a)) {
        PassArgs r = a;
        r.A = a.B;
        r.lda = a.ldb;
        r.B = a.A;
        r.ldb = a.lda;
        r.nops = 1;
        launch_triples(g, EPI_Y, r, a.nops, 1.0, part, s);
    } else {
        launch_pass(MODE_REDOPS, EPI_Y, a, s);
    }
}

// ---------------------------------------------------------------- outside ----
// Every record of the outside-space set against the product form, one thread
// per target: its label is the degree-6 string of its lexicographic rank, and
// its records are 20 (m - 6) different pairs (ascending), each I = U + q, J =
// V + q of a cut Q = U + V with factor c s(U, V) sigma(U, q) sigma(V, q).
__global__ void k_check_outside(int64_t n, int m, const uint32_t* bin, const uint64_t* labels, const uint64_t* olabels,
                                const int64_t* off, const uint2* rec, double c, int32_t* bad) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint64_t Q = olabels[k];
    bool ok = __popcll(Q) == 6 && off[k + 1] - off[k] == 20 * (m - 6) && (m == 64 || Q >> m == 0);
    int64_t rank = n - 1;
    int t = 6;
    for (uint64_t x = Q; ok && x; x &= x - 1) rank -= bin[t-- * 64 + m - 1 - (__ffsll((long long)x) - 1)];
    ok = ok && rank == k;
    uint64_t prev = 0;
    for (int64_t e = off[k]; ok && e < off[k + 1]; ++e) {
        const uint2 r = rec[e];
        const uint32_t i = r.x & 0xFFFFFFu, j = r.y & 0xFFFFFFu;
        const uint64_t I = labels[i], J = labels[j], both = I & J, U = I & ~both, V = J & ~both;
        const uint64_t key = (uint64_t)i << 32 | j;
        ok = (e == off[k] || key > prev) && __popcll(I) == 4 && __popcll(J) == 4 && __popcll(both) == 1 && (U ^ V) == Q;
        prev = key;
        int inv = 0;  // pairs u > v
        for (uint64_t v = V; v; v &= v - 1) inv += __popcll(U & ~((v & (~v + 1)) - 1));
        inv += __popcll(U & ~(both - 1)) + __popcll(V & ~(both - 1));
        const double f = (double)__builtin_bit_cast(float, (r.x & 0xFF000000u) | ((r.y >> 24) << 16));
        ok = ok && f == ((inv & 1) ? -c : c);
    }
    if (!ok) *bad = 1;
}

void build_outside(Graph& g, const HostGraph& hg) {
    TriPlan& p = g.tri;
    const int64_t n = g.n_out;
    const int m = p.m;
    p.release_outside();
    if (!p.ok || !g.have_outside || m < kOutMinModes || n < 1 || hg.off[2][1] == hg.off[2][0]) return;
    std::vector<uint32_t> bin(7 * 64);
    for (int k = 0; k < 7; ++k)
        for (int c = 0; c < 64; ++c) {
            double b = 1.0;
            for (int i = 0; i < k; ++i) b = b * (c - i) / (i + 1);
            bin[k * 64 + c] = c < k ? 0u : (uint32_t)std::llround(b);
        }
    if (n != (int64_t)bin[6 * 64 + m]) return;
    std::vector<uint32_t> pair2, tri3;
    for (int z = 1; z < m; ++z)
        for (int y = 0; y < z; ++y) pair2.push_back((uint32_t)(y | z << 8));
    for (int z = 2; z < m; ++z)
        for (int y = 1; y < z; ++y)
            for (int x = 0; x < y; ++x) tri3.push_back((uint32_t)(x | y << 8 | z << 16));
    // tiles for blocks of 16, 32 and 64 rows; the three-cut ones (three times the
    // steps) first
    std::vector<int4> tasks;
    for (int w = 0; w < 3; ++w) {
        const int rt = 16 << w;
        p.task0[w] = (int32_t)tasks.size();
        auto add = [&](int x, int rows, int cols) {
            for (int r = 0; r < rows; r += rt)
                for (int j = 0; j < cols; j += kTriW) tasks.push_back(make_int4(x, r, j, rows));
        };
        for (int a = 0; a < m; ++a)
            for (int e = a + 4; e < m; ++e)
                for (int f = e + 1; f < m; ++f) add(a | e << 8 | f << 16, (e - a - 1) * (e - a - 2) / 2, e - a - 1);
        for (int a = 0; a < m; ++a)
            for (int e = a + 4; e < m - 1; ++e) {
                const int d = e - a - 1;
                add(a | e << 8 | 1 << 24, d * (d - 1) * (d - 2) / 6, m - 1 - e);
            }
        p.task0[w + 1] = (int32_t)tasks.size();
    }
    upload(&p.bin, bin.data(), bin.size());
    upload(&p.pair2, pair2.data(), pair2.size());
    upload(&p.tri3, tri3.data(), tri3.size());
    upload(&p.tasks, tasks.data(), tasks.size());
    // the factor of the first record, the others against it
    const uint64_t Q0 = hg.out_labels[0];
    const uint64_t I = hg.labels[hg.ri[2][0]], J = hg.labels[hg.rj[2][0]], both = I & J, U = I & ~both, V = J & ~both;
    int inv = 0;
    for (uint64_t v = V; v; v &= v - 1) inv += __builtin_popcountll(U & ~((v & (~v + 1)) - 1));
    inv += __builtin_popcountll(U & ~(both - 1)) + __builtin_popcountll(V & ~(both - 1));
    if ((U ^ V) != Q0 || __builtin_popcountll(both) != 1) return;
    p.cout = (inv & 1) ? -(double)hg.rc[2][0] : (double)hg.rc[2][0];
    struct Temp {
        uint64_t *labels = nullptr, *out = nullptr;
        int32_t* bad = nullptr;
        ~Temp() {
            (void)hipFree(labels);
            (void)hipFree(out);
            (void)hipFree(bad);
        }
    } d;
    int32_t bad = 0;
    upload(&d.labels, hg.labels, (size_t)g.N);
    upload(&d.out, hg.out_labels, (size_t)n);
    upload(&d.bad, &bad, 1);
    hipLaunchKernelGGL(k_check_outside, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, 0, n, m, p.bin, d.labels, d.out,
                       g.csr[2][0].off, g.csr[2][0].rec, p.cout, d.bad);
    HIP_CHECK(hipMemcpy(&bad, d.bad, 4, hipMemcpyDeviceToHost));
    p.out_ok = p.cout != 0.0 && !bad;
}

// Partial rows of the outside-space products: 4 per target, for as many operands at a
// time as fit 2 GiB (0: not even one does).
size_t outside_least(const Graph& g, int64_t nsets) { return (size_t)(4 * g.n_out * nsets) * sizeof(double); }

// The products do 1.9 (24 modes) to 4 (16) times the records' operations on the
// padding of their tiles, and every tile is a chain of 3 m / 4 steps; the records are
// streamed once per column group of the segment kernel.  One action, us, segment
// kernel -> products (with the 4 us that putting their partial rows in order costs):
//   above the line  24 modes, 8 sets x 3 operands FP64 833 -> 302, 16 x 3 float 649 -> 438
//                   22 x 1 x 3 FP64 169 -> 136, 20 x 4 x 3 float 83 -> 71, 18 x 8 x 3 FP64 80 -> 74
//   below it        20 x 1 x 3 FP64 79 -> 86, 18 x 8 x 3 float 42 -> 56, 18 x 4 x 3 FP64 48 -> 61, 16 x 8 x 3 30 -> 46
static bool outside_faster(const Graph& g, int64_t nsets, bool f64) {
    return g.tri.m >= (nsets == 1 ? 22 : f64 && nsets > 4 ? 18 : 20);
}

size_t outside_partial_bytes(const Graph& g, int64_t nsets, int64_t nops) {
    constexpr size_t kCap = (size_t)2 << 30;
    // FP64's side of the line holds the floats', whose rows reach further
    if (!g.tri.out_ok || !outside_faster(g, nsets, true) || !tri_reach(g, nops * nsets, false)) return 0;
    const size_t one = outside_least(g, nsets);
    return one > kCap ? 0 : one * std::min<size_t>((size_t)nops, kCap / one);
}

bool outside_usable(const Graph& g, const PassArgs& a) {
    const bool f64 = a.precision == CUT_F64;
    return g.tri.out_ok && a.precision != CUT_F32 && outside_faster(g, a.nsets, f64) &&
           tri_reach(g, std::max(a.lda, a.ldb), f64);
}

void launch_outside(const Graph& g, const PassArgs& a, double* part, size_t bytes, hipStream_t s) {
    const TriPlan& p = g.tri;
    const bool f32 = a.precision != CUT_F64;
    const int64_t esz = f32 ? 4 : 8;
    const int sq = a.nsets <= 4 ? 1 : a.nsets <= 8 ? 2 : 4, w = sq == 4 ? 0 : sq == 2 ? 1 : 2;
    const int chunks = (a.nsets + 4 * sq - 1) / (4 * sq), ntask = p.task0[w + 1] - p.task0[w];
    const int fit = (int)std::min<size_t>((size_t)a.nops, bytes / outside_least(g, a.nsets));
    const int most = f32 ? tri_ops<float>() : tri_ops<double>();
    const int64_t bytesA = ((g.N - 1) * a.lda + a.nsets) * esz;
    const int64_t bytesB = ((g.N - 1) * a.ldb + (int64_t)a.nops * a.nsets) * esz;
    for (int o = 0; o < a.nops; o += fit) {
        const int nops = std::min(fit, (int)a.nops - o);
        TriArgs t{};
        t.tab = p.tab;
        t.m = p.m;
        t.nt = p.nt;
        t.ntau = p.ntau;
        t.ntp = p.ntp;
        t.N = g.n_out;
        t.lda = (int32_t)a.lda;
        t.ldb = (int32_t)a.ldb;
        t.nsets = a.nsets;
        t.s1 = a.nsets;
        t.nred = 1;
        t.ldp = (int64_t)nops * a.nsets;
        t.chunks = chunks;
        t.tasks = p.tasks + p.task0[w];
        t.bin = p.bin;
        t.pair2 = p.pair2;
        t.tri3 = p.tri3;
        t.A = a.A;
        t.bytesA = (uint32_t)bytesA;
        for (int q = 0; q < nops;) {
            const int left = nops - q, pieces = (left + most - 1) / most, k = (left + pieces - 1) / pieces;
            const int64_t bo = (int64_t)(o + q) * a.nsets * esz;
            t.B = (const char*)a.B + bo;
            t.bytesB = (uint32_t)(bytesB - bo);
            t.p4 = part + (int64_t)q * a.nsets;
            const dim3 grid((unsigned)((int64_t)ntask * chunks));
            if (f32) launch_outside_t<float>(t, k, sq, grid, s);
            else launch_outside_t<double>(t, k, sq, grid, s);
            q += k;
        }
        TriCombineArgs c{};
        c.p4 = part;
        c.nops = nops;
        c.nsets = a.nsets;
        c.w = a.nsets;
        c.N = g.n_out;
        c.ldp = t.ldp;
        c.c = p.cout;
        c.scale = a.scale;
        c.y = (double*)a.y + (int64_t)o * a.nsets;
        c.ldy = a.ldy;
        c.accumulate = a.accumulate;
        c.f32 = f32 ? 1 : 0;
        c.off = g.csr[2][0].off;
        c.rec = g.csr[2][0].rec;
        c.A = a.A;
        c.B = (const char*)a.B + (int64_t)o * a.nsets * esz;
        c.lda = a.lda;
        c.ldb = a.ldb;
        c.nred = 1;
        c.sign = 1.0;
        hipLaunchKernelGGL((k_tri_combine<EPI_Y>), dim3((unsigned)((g.n_out * t.ldp + 255) / 256)), dim3(256), 0, s, c, 0u);
    }
}

}  // namespace cut
